"""Quantizers: both sides of the column lengths at which the FP8 kernel or its
number of loads changes, and the BF16 one's pads and cache rule, byte for byte
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_quantize import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,lda,ldo", [
    (3, 4, 256), (60, 60, 64), (61, 64, 68), (255, 256, 256), (253, 256, 260), (256, 256, 512), (509, 512, 512), (510, 512, 516),
    (512, 512, 1024), (1023, 1024, 1024), (1024, 1024, 1028), (1027, 1028, 2048)])
def test_loads_per_wave(gpu, m, lda, ldo):
    n = 11
    A = _inputs(m, n, lda, m + ldo)
    dA = torch.from_numpy(A).cuda()
    out = torch.full((n, ldo), 0xAB, dtype=torch.uint8, device="cuda")
    sc = torch.full((n,), -1.0, device="cuda")
    gpu.quantize(dA.data_ptr(), m, n, lda, gpu.FP8_E4M3, out.data_ptr(), ldo, sc.data_ptr())
    codes, scl = oracle.quantize_fp8(np.ascontiguousarray(A[:, :m]), m, ldo=ldo)
    ok = scl > 0  # (a column whose scale underflows to zero has no defined codes)
    assert np.array_equal(sc.cpu().numpy().view(np.int32), scl.astype(np.float32).view(np.int32))
    assert np.array_equal(out.cpu().numpy()[ok], codes[ok])


@pytest.mark.parametrize("m,n,lda,ldo", [
    (1, 13, 4, 264), (4, 13, 4, 8), (5, 13, 8, 256), (12, 13, 12, 256),  # mostly pads
    (2100, 22000, 2100, 2304),                                          # past the caches
])
def test_bf16_pads_and_large(gpu, m, n, lda, ldo):
    A = _inputs(m, n, lda, m + ldo) if n < 100 else np.random.default_rng(1).standard_normal((n, lda)).astype(np.float32)
    out = torch.full((n, ldo), 0x5A5A, dtype=torch.int16, device="cuda")
    dA = torch.from_numpy(A).cuda()
    gpu.quantize(dA.data_ptr(), m, n, lda, gpu.BF16, out.data_ptr(), ldo, None)
    want = oracle.quantize_bf16(np.ascontiguousarray(A[:, :m]), m, ldo=ldo)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), want.view(np.uint16))
