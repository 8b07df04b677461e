"""The step of a small explicit target in one workgroup: both sides of its limits
(rows, target columns, picks), remainders of its columns in flight and of its
wave-sized row groups, each storage and target type, and columns it has to
reject.  Each against the general kernels (GCSS_CHAIN=0): the same picks on
planted inputs, objectives to FP64 rounding, and a basis orthonormal to FP64
rounding."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import colstore32

pytestmark = pytest.mark.gpu


def _run(gpu, A, B, m, k, r, monkeypatch, general, scales=None):
    if general:
        monkeypatch.setenv("GCSS_CHAIN", "0")
    else:
        monkeypatch.delenv("GCSS_CHAIN", raising=False)
    s = gpu.Selector(A, m, k_max=k, r_max=r, self_target=False, scales=scales)
    s.set_target(B)
    idx, obj, ns, _ = s.select(k)
    Q = s.read(gpu.STATE_Q, m * ns, np.float64).reshape(ns, m)
    s.close()
    return np.asarray(idx), np.asarray(obj), ns, Q


def _target(A, pos, r, dtype):
    rng = np.random.default_rng(r)
    B = np.zeros((r, (A.shape[0] + 63) // 64 * 64), np.float32)
    B[:, :A.shape[0]] = (A[:, pos] @ rng.standard_normal((len(pos), r)) / np.sqrt(r)).T
    return torch.as_tensor(B, device="cuda").to(dtype)


def _equal(a, b, k):
    assert a[2] == b[2] == k
    np.testing.assert_array_equal(a[0], b[0])
    assert np.max(np.abs(a[1] - b[1])) <= 1e-12 * a[1][0]
    # both orthogonalise twice: FP64 rounding of k-term sums, a few ulps
    for Q in (a[3], b[3]):
        assert np.max(np.abs(Q @ Q.T - np.eye(k))) <= 2e-14
    assert np.max(np.abs(a[3] - b[3])) <= 1e-12


@pytest.mark.parametrize("m,n,r,k", [
    (24, 300, 8, 8),
    (65, 403, 17, 19),
    (512, 1500, 64, 32),   # the largest
    (513, 1500, 64, 32),   # a row more, a column more, a pick more: the slab form
    (512, 1500, 65, 32),
    (512, 1500, 64, 33),
    (333, 70000, 33, 17),  # more winners than the workgroup has threads in a wave
])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_one_workgroup_equals_general(gpu, monkeypatch, m, n, r, k, dtype):
    A, pos = synth.planted_dense(m, n, k, 1.05, seed=m + r + k)
    A32 = torch.as_tensor(colstore32(A), device="cuda")
    B = _target(A, pos, r, dtype)
    _equal(*(_run(gpu, A32, B, m, k, r, monkeypatch, g) for g in (False, True)), k)


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
def test_quantised_columns(gpu, monkeypatch, fmt):
    m, n, r, k = 130, 900, 20, 20
    A, pos = synth.planted_dense(m, n, k, 1.3, seed=5)
    Aq, sc = gpu.quantize_tensor(torch.as_tensor(colstore32(A), device="cuda"), m, fmt)
    B = _target(A, pos, r, torch.float32)
    _equal(*(_run(gpu, Aq, B, m, k, r, monkeypatch, g, sc) for g in (False, True)), k)


def test_rejected_columns(gpu, monkeypatch):
    # columns of a 12-dimensional space: the thirteenth pick has none left
    m, n, r, k = 40, 200, 16, 16
    A12, pos = synth.planted_dense(12, n, 8, 1.3, seed=9)
    A = np.zeros((m, n), A12.dtype)
    A[:12] = A12
    A32 = torch.as_tensor(colstore32(A), device="cuda")
    B = _target(A, pos, r, torch.float32)
    a, b = (_run(gpu, A32, B, m, k, r, monkeypatch, g) for g in (False, True))
    assert a[2] == b[2] and 8 <= a[2] <= 12
    np.testing.assert_array_equal(a[0][:8], b[0][:8])
    assert np.max(np.abs(a[1][:9] - b[1][:9])) <= 1e-12 * a[1][0]
