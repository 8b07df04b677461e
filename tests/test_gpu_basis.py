"""Reconstruction error of a caller's subset: the all-at-once basis (chunks of
128 columns) at its sizes' edges, and the subsets it hands back to
Gram-Schmidt, against FP64 QR on the CPU."""
import numpy as np
import pytest

import synth
from tests.gpu_util import colstore32, dev, stored_dense

pytestmark = pytest.mark.gpu


def _ref(Av, B, idx):
    """Basis of the columns idx that are independent, and the target's error."""
    Q, R = np.linalg.qr(Av[:, idx])
    Q = Q * np.sign(np.diag(R))
    T = Av if B is None else B
    return Q, float(np.sum((T - Q @ (Q.T @ T)) ** 2))


@pytest.mark.parametrize("m,n,k,r,dt", [
    (65, 300, 8, 5, "f32"),       # the smallest subset taken all at once
    (100, 400, 7, 5, "f32"),      # one fewer: Gram-Schmidt
    (333, 700, 127, 16, "f32"), (333, 700, 128, 16, "bf16"), (333, 700, 129, 16, "f32"),
    (130, 600, 130, 0, "f32"),    # k = m, two chunks, B = A
    (1000, 900, 300, 20, "fp8"),  # three chunks
    (2050, 600, 260, 0, "f32"),
    (8192, 400, 40, 12, "f32"),
])
def test_subset_error_and_basis(gpu, m, n, k, r, dt):
    rng = np.random.default_rng(m + k)
    A32 = colstore32(rng.standard_normal((m, n)) * np.exp(rng.standard_normal((1, n))))
    if dt == "f32":
        A, sc, Av = dev(A32), None, stored_dense(A32, m)
    else:
        A, sc = gpu.quantize_tensor(dev(A32), m, dt)
        import torch
        t = A.view(torch.bfloat16) if dt == "bf16" else A.view(torch.float8_e4m3fn)
        Av = t.float().cpu().numpy()[:, :m].T.astype(np.float64)
        if sc is not None:
            Av = Av * sc.cpu().numpy().astype(np.float64)[None, :]
    s = gpu.Selector(A, m, k_max=k, r_max=max(r, 1), self_target=r == 0, scales=sc)
    B = None
    if r:
        Bs = colstore32(rng.standard_normal((m, r)))
        s.set_target(dev(Bs))
        B = stored_dense(Bs, m)
    else:
        s.set_target(None)
    idx = rng.permutation(n)[:k]
    err = s.reconstruction_error(idx)
    Q = s.read(gpu.STATE_Q, m * k, np.float64).reshape(k, m).T
    Qr, er = _ref(Av, B, idx)
    norm = float(np.sum((Av if B is None else B) ** 2))
    assert np.max(np.abs(Q.T @ Q - np.eye(k))) <= 2e-14
    # the two bases differ by their factorisations' rounding, eps * cond of the
    # subset (Gaussian columns of norms e^{+-3}: < 1e6 up to k = m), squared
    # away in the error
    cond = np.linalg.cond(Av[:, idx] / np.linalg.norm(Av[:, idx], axis=0))
    assert np.max(np.abs(Q - Qr)) <= 1e-13 * cond
    assert abs(err - er) <= 1e-12 * norm
    s.close()


def _gram_schmidt(C):
    """Basis by the library's rule: a column whose residual's squared norm is at
    most 1e-13 of its own adds nothing."""
    Q = np.zeros((C.shape[0], 0))
    for a in C.T:
        e = a - Q @ (Q.T @ a)
        e -= Q @ (Q.T @ e)
        if e @ e > 1e-13 * (a @ a):
            Q = np.column_stack([Q, e / np.sqrt(e @ e)])
    return Q


def test_dependent_columns_are_left_to_gram_schmidt(gpu):
    """A repeated direction, a zero column and a nearly dependent column: the
    error is that of the independent ones."""
    m, n = 300, 200
    rng = np.random.default_rng(5)
    A = rng.standard_normal((m, n))
    A[:, 3] = 2.0 * A[:, 1]
    A[:, 7] = 0.0
    A[:, 9] = A[:, 2] + 1e-6 * A[:, 4]
    A32 = colstore32(A)
    Av = stored_dense(A32, m)
    Bs = colstore32(rng.standard_normal((m, 9)))
    s = gpu.Selector(dev(A32), m, k_max=20, r_max=9)
    s.set_target(dev(Bs))
    B = stored_dense(Bs, m)
    for idx in ([1, 3] + list(range(20, 30)), [7] + list(range(20, 32)), list(range(10)) + [50]):
        err = s.reconstruction_error(np.array(idx))
        Q = _gram_schmidt(Av[:, idx])
        want = float(np.sum((B - Q @ (Q.T @ B)) ** 2))
        # (a nearly dependent direction is resolved to eps / 1e-6)
        assert abs(err - want) <= 1e-8 * float(np.sum(B ** 2)), idx
    s.close()
