"""Selections whose threshold lets in columns that are dependent but for a small
part: the basis is orthonormal to FP64 rounding.  For a part of 1e-12 that takes
two projections in FP64 (a first one of binary32 coefficients leaves 1e-7 of the
column, whose FP64 rounding is 1e-11 of that part); from tau = 1e-6 on, where the
first one takes them, the parts are twice the smallest that is accepted."""
import numpy as np
import pytest

from tests.gpu_util import colstore32, dev

pytestmark = pytest.mark.gpu


def _near_copies(m, n, part):
    """Integer multiples (of different rounding each) of one column of small
    integers, exact in binary32, each with an entry of `part` of its norm in a
    row of its own."""
    rng = np.random.default_rng(m + n)
    h = m // 2
    A = np.zeros((m, n))
    A[:h] = rng.integers(-100, 101, (h, 1)) * rng.integers(50, 1000, (1, n))
    A[h + np.arange(n), np.arange(n)] = part * np.linalg.norm(A[:h], axis=0)
    return A


@pytest.mark.parametrize("tau,part", [(1e-28, 1e-12), (9e-7, 2e-3), (1e-6, 2e-3), (0.0, 2e-2)])
@pytest.mark.parametrize("m,r", [
    (300, 0), (300, 20), (300, 130),  # the chain's forms: slab on C, one workgroup, slab
    (4096, 500)])                     # and without the slab's partials
def test_basis_of_nearly_dependent_picks(gpu, m, r, tau, part):
    n, k = 100, 24
    A = _near_copies(m, n, part)
    s = gpu.Selector(dev(colstore32(A)), m, k_max=k, r_max=r, self_target=r == 0, tau=tau)
    s.set_target(dev(colstore32(np.random.default_rng(r).standard_normal((m, r)))) if r else None)
    idx, obj, ns, _ = s.select(k)
    assert ns >= 4  # (of 1e-12, half of the copies or so keep a residual above zero in rounding)
    Q = s.read(gpu.STATE_Q, m * ns, np.float64).reshape(ns, m)
    assert np.max(np.abs(Q @ Q.T - np.eye(ns))) <= 2e-14
    s.close()
