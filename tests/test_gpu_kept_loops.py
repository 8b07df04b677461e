"""The captured loops that a context keeps when B = A is set again: they follow
the embedding's buffer and its row stride, and they read A's values as they
are at the call."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import colstore32, dev, stored_dense

pytestmark = pytest.mark.gpu


def _selector(gpu, m, n, k, seed):
    A32 = colstore32(synth.gauss_lowrank_dense(m, n, 20, 0.05, seed=seed))
    s = gpu.Selector(dev(A32), m, k_max=k, self_target=True)
    s.set_target(None)
    return s, stored_dense(A32, m)


def _check_rows(s, gpu, W, Av, m, n, k):
    """W's rows are Q^T A (a binary32 store of FP64 dots), its pads untouched."""
    Q = s.read(gpu.STATE_Q, m * k, np.float64).reshape(k, m)
    Wh = W.cpu().numpy()
    assert np.all(Wh[:, n:] == 7.0)
    norms = np.sqrt(np.sum(Av * Av, axis=0))
    assert np.max(np.abs(Wh[:, :n] - Q @ Av) / norms[None, :]) <= 1e-6


@pytest.mark.parametrize("again", [True, False])
@pytest.mark.parametrize("path", ["sync", "async"])
def test_embedding_stride_changes_on_one_buffer(gpu, path, again):
    """One buffer, three strides, growing and shrinking: every selection writes
    W with the stride that was set last and nothing outside its rows."""
    m, n, k = 120, 900, 9
    s, Av = _selector(gpu, m, n, k, seed=3)
    buf = torch.empty(k * (n + 64), dtype=torch.float32, device="cuda")
    out = s.select_async(k)
    for ldw in (n + 1, n + 64, n):
        buf.fill_(7.0)
        W = buf[:k * ldw].view(k, ldw)
        s.set_embedding(W)
        if again:
            s.set_target(None)
        if path == "sync":
            s.select(k)
        else:
            s.select_async(k, out)
            torch.cuda.synchronize()
        _check_rows(s, gpu, W, Av, m, n, k)
        assert torch.all(buf[k * ldw:] == 7.0)
    s.close()


@pytest.mark.parametrize("path", ["sync", "async"])
def test_same_target_again_after_a_changes(gpu, path):
    """A overwritten in place and B = A set again: the results of a context
    made for the new values."""
    m, n, k = 200, 1100, 8
    s, _ = _selector(gpu, m, n, k, seed=4)
    out = s.select_async(k)
    first = s.select(k)
    A2 = colstore32(synth.planted_dense(m, n, k, 1.4, seed=5)[0])
    s.A.copy_(torch.from_numpy(A2))
    s.set_target(None)
    if path == "sync":
        idx, obj, ns, _ = s.select(k)
    else:
        s.select_async(k, out)
        idx, obj, ns = (t.cpu().numpy() for t in out)
        ns = int(ns[0])
    t = gpu.Selector(dev(A2), m, k_max=k, self_target=True)
    t.set_target(None)
    want = t.select(k)
    assert ns == want[2] == k
    np.testing.assert_array_equal(idx, want[0])
    np.testing.assert_array_equal(np.asarray(obj).view(np.int64), np.asarray(want[1]).view(np.int64))
    assert not np.array_equal(first[0], idx)
    s.close()
    t.close()
