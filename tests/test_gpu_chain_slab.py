"""The chain's forms at the sizes where one gives way to another: the slab form
(partials per 32 rows) up to its limit on rows x (r + k), the dot kernels
above it, the columns per thread (4, 8 and 16 times 32, then further rounds),
and a problem whose history of omega is not kept.  Each against the general
kernels (GCSS_CHAIN=0): the same picks on planted inputs, objectives to FP64
rounding, and a basis orthonormal to FP64 rounding."""
import os

import numpy as np
import pytest

import synth
from tests.gpu_util import colstore32, dev

pytestmark = pytest.mark.gpu


def _run(gpu, A, m, k, monkeypatch, *, general, B=None, r=0):
    if general:
        monkeypatch.setenv("GCSS_CHAIN", "0")
    else:
        monkeypatch.delenv("GCSS_CHAIN", raising=False)
    s = gpu.Selector(A, m, k_max=k, r_max=r, self_target=B is None)
    s.set_target(B)
    idx, obj, ns, _ = s.select(k)
    Q = s.read(gpu.STATE_Q, m * ns, np.float64).reshape(ns, m)
    s.close()
    return np.asarray(idx), np.asarray(obj), ns, Q


@pytest.mark.parametrize("m,n,r,k", [
    (33, 400, 16, 20),        # two row groups, the second of one row
    (512, 1500, 128, 128),    # 4 columns per thread, full
    (512, 1500, 129, 129),    # 8
    (544, 1500, 257, 40),     # 16 for the target
    (1025, 1500, 0, 60),      # B = A
    (4096, 900, 344, 40),     # 128 row groups x 384: the slab form's largest
    (4096, 900, 345, 40),     # one more: dot kernels
    (600, 1400, 513, 30),     # more target columns than one round
    (640, 1600, 24, 520),     # more picks than one round
    (60, 300000, 16, 20),     # history of omega larger than it may be
])
def test_chain_forms_equal_general(gpu, monkeypatch, m, n, r, k):
    ratio = 1.05 if k <= 150 else 1.01
    A, pos = synth.planted_dense(m, n, k, ratio, seed=m + r + k)
    A32 = dev(colstore32(A))
    B = None
    if r:
        rng = np.random.default_rng(r)
        ldb = (m + 63) // 64 * 64
        Bd = np.zeros((r, ldb), np.float32)
        Bd[:, :m] = (A[:, pos] @ rng.standard_normal((k, r)) / np.sqrt(r)).T
        B = dev(Bd)
    a = _run(gpu, A32, m, k, monkeypatch, general=False, B=B, r=r)
    b = _run(gpu, A32, m, k, monkeypatch, general=True, B=B, r=r)
    assert a[2] == b[2] == k
    np.testing.assert_array_equal(a[0], b[0])
    assert np.max(np.abs(a[1] - b[1])) <= 1e-12 * a[1][0]
    # both orthogonalise twice: FP64 rounding of k-term sums, a few ulps
    for Q in (a[3], b[3]):
        assert np.max(np.abs(Q @ Q.T - np.eye(k))) <= 2e-14
    assert np.max(np.abs(a[3] - b[3])) <= 1e-12
