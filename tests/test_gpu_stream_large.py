"""The streaming pass of a matrix larger than the last-level cache (its results
held in LDS and written in bursts): scores, residual norms and embedding rows
against FP64 products on the same stored values, ragged rows and columns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("target", ["explicit", "self"])
@pytest.mark.parametrize("dt,m,n,upw", [("f32", 1003, 70001, 4), ("f32", 1003, 140001, 64),  # the buffer overflows
                                        ("bf16", 1003, 140001, 4), ("fp8", 2001, 140003, 4)])
def test_large_pass_against_fp64(gpu, dt, m, n, upw, target):
    gen = torch.Generator(device="cuda").manual_seed(n)
    lda = (m + 15) // 16 * 16
    A32 = torch.randn(n, lda, generator=gen, device="cuda")
    A32 *= torch.exp(0.5 * torch.randn(n, 1, generator=gen, device="cuda"))
    A32[:, m:] = 0.0
    A, sc = (A32, None) if dt == "f32" else gpu.quantize_tensor(A32, m, dt)
    assert A.numel() * A.element_size() > 256 << 20
    view = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dt]
    k, r = 4, 24
    s = gpu.Selector(A, m, k_max=k, r_max=r, self_target=target == "self", scales=sc)
    s.tuning(stream_upw=upw)
    B = None
    if target == "explicit":
        B = torch.zeros(r, (m + 3) // 4 * 4, device="cuda")
        B[:, :m] = torch.randn(r, m, generator=gen, device="cuda")
    s.set_target(B)
    W = torch.full((k, n + 3), 7.0, device="cuda")
    s.set_embedding(W)
    assert s.select(k)[2] == k
    # (the pass after the last pick writes its row of W only)
    Q = torch.from_numpy(s.read(gpu.STATE_Q, m * k, np.float64).reshape(k, m)).cuda()
    f = torch.from_numpy(s.read(gpu.STATE_F, n, np.float64)).cuda()
    g = torch.from_numpy(s.read(gpu.STATE_G, n, np.float64)).cuda()
    if B is None:
        C = torch.zeros(m, m, dtype=torch.float64, device="cuda")
    for pass_ in range(2):
        for c in range(0, n, 20000):
            e = min(n, c + 20000)
            Ac = A[c:e].view(view).float().double()[:, :m]
            if sc is not None:
                Ac = Ac * sc[c:e].double()[:, None]
            if pass_ == 0:
                if B is None:
                    C += Ac.T @ Ac
                continue
            w = Ac @ Q.T
            E = Ac - w[:, :k - 1] @ Q[:k - 1]
            n2 = (Ac * Ac).sum(1)
            fx = ((E @ C) * E).sum(1) if B is None else ((E @ B[:, :m].double().T) ** 2).sum(1)
            f0 = ((Ac @ C) * Ac).sum(1) if B is None else ((Ac @ B[:, :m].double().T) ** 2).sum(1)
            # binary32 dots of m terms: sqrt(m) 2^-24 of the norms at most, with a margin
            assert torch.max((W[:, c:e].T.double() - w).abs() / n2.sqrt()[:, None]) <= 1e-5
            assert torch.max((g[c:e] - (E * E).sum(1)).abs() / n2) <= 1e-5
            assert torch.max((f[c:e] - fx).abs() / f0) <= 1e-4
    assert torch.all(W[:, n:] == 7.0)
    s.close()
