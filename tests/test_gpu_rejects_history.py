"""Rejected picks in the chain's forms that read the history of omega (tau >=
1e-6): near copies of the best column whose exact residual is 0.998 tau, which
the binary32 dot products behind their tracked one leave candidates or not.
The picks are the oracle's, whose FP64 scores see the residual exactly."""
import math

import numpy as np
import pytest

import oracle
from tests.gpu_util import colstore32, dev, f64cs, stored_dense

pytestmark = pytest.mark.gpu

TAU = 1e-6


def _case(m, n, r):
    """B = X diag(sqrt(s2)) Y^T; column 10 is 3 v, v = (x1 + x2) / sqrt(2), the
    best; columns 1100..1139 are c (v - a w), w = (x1 - x2) / sqrt(2), with
    a^2 / (1 + a^2) = 0.998 tau; ten columns x3 .. x12 over a 1e-3 noise."""
    rng = np.random.default_rng(m + r)
    X, _ = np.linalg.qr(rng.standard_normal((m, r)))
    Y, _ = np.linalg.qr(rng.standard_normal((r, r)))
    B = X @ np.diag(np.sqrt([2.0, 1.0] + [0.8 * 0.75 ** j for j in range(r - 2)])) @ Y.T
    v, w = (X[:, 0] + X[:, 1]) / math.sqrt(2), (X[:, 0] - X[:, 1]) / math.sqrt(2)
    A = 1e-3 * rng.standard_normal((m, n)) / math.sqrt(m)
    A[:, 10] = 3.0 * v
    near = list(range(1100, 1140))
    for j in near:
        A[:, j] = rng.uniform(1.5, 4.5) * (v - math.sqrt(0.998 * TAU) * w)
    planted = [50, 120, 300, 777, 900, 1010, 1200, 1500, 1700, 1900]
    A[:, planted] = X[:, 2:12]
    return A, B, near, planted


@pytest.mark.parametrize("m,kmax,r", [
    (512, 10, 16),      # one workgroup
    (4096, 10, 16),     # slab
    (8192, 200, 200)])  # without its partials
def test_rejected_picks_with_the_history(gpu, m, kmax, r):
    n, k = 2000, 10
    A, B, near, planted = _case(m, n, r)
    A32, B32 = colstore32(A), colstore32(B)
    ref = oracle.select(f64cs(stored_dense(A32, m)), m, k, B=f64cs(stored_dense(B32, m)), tau=TAU)
    assert list(ref["idx"]) == [10] + planted[:k - 1] and np.min(ref["gap"]) > 1e-4
    s = gpu.Selector(dev(A32), m, k_max=kmax, r_max=r, tau=TAU)
    s.set_target(dev(B32))
    for _ in range(2):  # captured, then replayed
        idx, obj, ns, st = s.select(k)
        fl = s.flags()
        assert fl["rejected"] > 0 and ns == k and st == gpu.OK and fl["finished"]
        assert list(idx) == list(ref["idx"])
        np.testing.assert_allclose(obj, ref["obj"], rtol=1e-5)
    d_idx, d_obj, d_ns = s.select_async(k)
    na, fa = int(d_ns.cpu()[0]), s.flags()
    assert na == k if fa["finished"] else fa["rejected"] >= gpu.ASYNC_SPARE_STEPS
    assert list(d_idx.cpu().numpy()[:na]) == list(idx[:na])
    assert np.array_equal(d_obj.cpu().numpy()[:na + 1], obj[:na + 1])
    s.close()
