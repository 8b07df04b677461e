"""Basis of a given subset of more than 128 columns (two chunks): a column of
the second chunk that depends on the first one is dropped by the same rule as
anywhere else (residual's squared norm at most 1e-13 of its own), so the error
does not depend on its place in the subset."""
import numpy as np
import pytest

from tests.gpu_util import colstore32, dev, stored_dense
from tests.test_gpu_basis import _gram_schmidt

pytestmark = pytest.mark.gpu

K = 140


def _columns(m, kind):
    """K columns, the last of which is the special one, and a target with
    energy in the direction that it would add."""
    rng = np.random.default_rng(m)
    if kind == "sparse":
        # exact arithmetic: unit vectors, then e_0 + 1e-7 e_200
        A = np.zeros((m, K))
        A[np.arange(K - 1), np.arange(K - 1)] = 1.0
        A[0, K - 1] = 1.0
        A[200, K - 1] = 1e-7
        B = rng.standard_normal((m, 6))
        B[200] *= 10.0
        return A, B
    A = rng.standard_normal((m, K)) * np.exp(rng.standard_normal((1, K)))
    if kind == "multiple":
        A[:, -1] = 1.7 * A[:, 2]  # stored rounded: off by 3e-8 of its norm
    elif kind == "near":
        A[:, -1] = A[:, 2] + 1e-5 * A[:, -1]  # kept: 1e-10 of its squared norm
    elif kind == "zero":
        A[:, -1] = 0.0
    elif kind == "nan":
        A[m // 2, -1] = np.nan
    elif kind == "inf":
        A[m // 2, -1] = np.inf
    return A, rng.standard_normal((m, 6))


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("m,kind", [
    (300, "sparse"), (4096, "sparse"), (300, "multiple"), (8192, "multiple"), (300, "near"),
    (4096, "near"), (300, "zero"), (300, "nan"), (300, "inf")])
def test_dependent_column_of_the_second_chunk(gpu, m, kind):
    A, B = _columns(m, kind)
    A32, B32 = colstore32(A), colstore32(B)
    Av, Bv = stored_dense(A32, m), stored_dense(B32, m)
    s = gpu.Selector(dev(A32), m, k_max=K, r_max=B.shape[1])
    s.set_target(dev(B32))
    last = np.arange(K)
    for idx in (last, np.roll(last, 20)):  # the special column last, and among the first 128
        Q = _gram_schmidt(Av[:, idx])
        assert Q.shape[1] == (K if kind == "near" else K - 1)
        want = float(np.sum((Bv - Q @ (Q.T @ Bv)) ** 2))
        # a direction of 1e-5 of its column is resolved to eps / 1e-5 = 2e-11
        assert abs(s.reconstruction_error(idx) - want) <= 1e-9 * float(np.sum(Bv ** 2))
    s.close()
