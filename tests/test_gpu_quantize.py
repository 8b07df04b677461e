"""Quantizer dispatch: the wide kernels (one and four waves per column) and the
element-wise one, at their sizes' edges and on the encoders' edge values, byte
for byte against the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _inputs(m, n, lda, seed):
    """Normal columns, code midpoints one ulp to each side, a wide range of
    column magnitudes (down to scales that underflow), zero columns."""
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((n, lda)).astype(np.float32)
    kind = np.arange(n) % 4
    mid = (rng.integers(-3584, 3585, size=(n, lda)) / 8.0).astype(np.float32) * rng.integers(1, 64, size=(n, 1))
    mid = (mid.astype(np.float32).view(np.int32) + rng.integers(0, 2, size=(n, lda), dtype=np.int32)).view(np.float32)
    A = np.where((kind == 1)[:, None], mid, A)
    mag = np.exp2(rng.integers(-140, 100, size=(n, 1)).astype(np.float32))
    A = np.where((kind == 2)[:, None], A * mag, A).astype(np.float32)
    A[kind == 3, ::3] = 0.0
    A[n // 2] = 0.0
    A[:, m:] = 9.0  # pads of A are never read into results
    return A


@pytest.mark.parametrize("m,lda,ldo", [
    (1, 4, 4), (63, 64, 64), (333, 336, 512),
    (2047, 2048, 2048), (2048, 2048, 2048),   # the most one wave holds
    (2049, 2052, 2056), (8192, 8192, 8192),   # four waves
    (8193, 8196, 8200),                       # element-wise: more than four waves hold
    (100, 101, 128), (100, 104, 101),         # element-wise: unaligned columns, odd output
])
def test_wide_and_general_kernels_match_the_oracle(gpu, m, lda, ldo):
    import torch
    n = 13
    A = _inputs(m, n, lda, m + ldo)
    dA = torch.from_numpy(A).cuda()
    src = np.ascontiguousarray(A[:, :m])
    out = torch.full((n, ldo), 0xAB, dtype=torch.uint8, device="cuda")
    sc = torch.full((n,), -1.0, device="cuda")
    gpu.quantize(dA.data_ptr(), m, n, lda, gpu.FP8_E4M3, out.data_ptr(), ldo, sc.data_ptr())
    codes, scl = oracle.quantize_fp8(src, m, ldo=ldo)
    # (a column whose scale underflows to zero has no defined codes)
    ok = scl > 0
    assert np.array_equal(sc.cpu().numpy().view(np.int32), scl.astype(np.float32).view(np.int32))
    assert np.array_equal(out.cpu().numpy()[ok], codes[ok])
    out = torch.full((n, ldo), 0x5A5A, dtype=torch.int16, device="cuda")
    gpu.quantize(dA.data_ptr(), m, n, lda, gpu.BF16, out.data_ptr(), ldo, None)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), oracle.quantize_bf16(src, m, ldo=ldo).view(np.uint16))


def test_non_finite_values_follow_the_encoder(gpu):
    """NaN keeps its sign with code 0x7F; an infinite column maximum makes an
    infinite scale, so finite entries get code 0."""
    import torch
    A = np.ones((3, 64), np.float32)
    A[0, 5], A[0, 6] = np.nan, np.copysign(np.nan, -1)
    A[1, 7] = np.inf
    A[2, 9] = -3.0
    codes, sc = gpu.quantize_tensor(torch.from_numpy(A).cuda(), 64, "fp8")
    c = codes.cpu().numpy()
    assert c[0, 5] == 0x7F and c[0, 6] == 0xFF and c[0, 0] == 0x7E
    assert np.isinf(sc.cpu().numpy()[1]) and c[1, 0] == 0 and (c[1, 7] & 0x7F) == 0x7F
    assert c[2, 9] == 0xFE
