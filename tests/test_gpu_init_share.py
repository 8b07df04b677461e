"""Initial scores where few columns share their row chunks between workgroups
(and right above), for both kernels and targets, against FP64."""
import numpy as np
import pytest

from tests.gpu_util import colstore32, dev, stored_dense

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,r", [
    (500, 1000, 0), (65, 130, 0), (1100, 4096, 0), (1100, 4097, 0),  # binary32 kernel, both tilings
    (600, 1024, 0), (2100, 3000, 0), (300, 40000, 0),                 # BF16-split kernel, B = A
    (520, 700, 130), (700, 1500, 300), (700, 1500, 513), (300, 3000, 100), (300, 34000, 300),
])
def test_initial_scores_match_fp64(gpu, m, n, r):
    rng = np.random.default_rng(m + n + r)
    A32 = colstore32(rng.standard_normal((m, 12)) @ rng.standard_normal((12, n)) + rng.standard_normal((m, n)))
    Av = stored_dense(A32, m)
    s = gpu.Selector(dev(A32), m, k_max=8, r_max=max(r, 1), self_target=r == 0)
    if r:
        Bs = colstore32(rng.standard_normal((m, r)))
        s.set_target(dev(Bs))
        want = np.sum((stored_dense(Bs, m).T @ Av) ** 2, axis=0)
    else:
        s.set_target(None)
        want = np.sum((Av @ Av.T @ Av) * Av, axis=0)
    f, g = s.read(gpu.STATE_F0, n, np.float64), s.read(gpu.STATE_G0, n, np.float64)
    # FP32 matrix-core dot products over a few thousand terms; FP64 norms
    assert np.max(np.abs(f - want) / want) <= 1e-4
    np.testing.assert_allclose(g, np.sum(Av * Av, axis=0), rtol=1e-12)
    s.close()
