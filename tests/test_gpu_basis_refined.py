"""Basis of a given subset of strongly correlated columns (a common direction
and a part d of their own): past what one orthonormalisation certifies, within
what a second one does, and beyond both.  Against Gram-Schmidt in FP64."""
import numpy as np
import pytest

from tests.gpu_util import colstore32, dev, stored_dense
from tests.test_gpu_basis import _gram_schmidt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3e-2, 3e-3, 5e-4, 2e-5, 1e-7])
@pytest.mark.parametrize("m,k,r", [(60, 60, 0), (200, 17, 5), (700, 128, 9), (700, 150, 9), (900, 300, 0)])
def test_correlated_columns(gpu, m, k, r, d):
    rng = np.random.default_rng(m + k)
    A = rng.standard_normal((m, 1)) + d * rng.standard_normal((m, k + 20))
    A *= np.exp(rng.standard_normal((1, k + 20)))
    A32 = colstore32(A)
    Av = stored_dense(A32, m)
    s = gpu.Selector(dev(A32), m, k_max=k, r_max=max(r, 1), self_target=r == 0)
    T = Av
    if r:
        B32 = colstore32(rng.standard_normal((m, r)))
        T = stored_dense(B32, m)
        s.set_target(dev(B32))
    else:
        s.set_target(None)
    idx = rng.permutation(k + 20)[:k]
    err = s.reconstruction_error(idx)
    C = Av[:, idx]
    want_q = _gram_schmidt(C)
    # (d = 1e-7: near the rule's 1e-13, as binary32 leaves it; any number stays)
    kb = k if d > 1e-6 else int(s.flags()["picks"])
    assert kb == want_q.shape[1] or d < 1e-6
    Q = s.read(gpu.STATE_Q, m * kb, np.float64).reshape(kb, m)
    assert np.max(np.abs(Q @ Q.T - np.eye(kb))) <= 2e-14
    if d > 1e-6:
        # spans agree to rounding times the condition of the scaled columns
        cond = np.linalg.cond(C / np.linalg.norm(C, axis=0))
        want = float(np.sum((T - want_q @ (want_q.T @ T)) ** 2))
        assert abs(err - want) <= 1e-14 * k * cond * float(np.sum(T ** 2))
    s.close()
