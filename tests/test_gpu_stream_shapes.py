"""The streaming passes at both sides of every row count where the rows per lane
or the waves per column change, for each storage type, target and load depth:
embedding rows against FP64, and the batched pass against the same columns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = [1, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192]


@pytest.mark.parametrize("dt", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("m", ROWS)
def test_every_shape_has_its_kernel(gpu, dt, m):
    n, r = 300, 5
    k = 1 if m == 1 else 3
    gen = torch.Generator(device="cuda").manual_seed(m)
    A = torch.randn(n, (m + 15) // 16 * 16, generator=gen, device="cuda")
    sc = None
    if dt != "f32":
        A, sc = gpu.quantize_tensor(A, m, dt)
    Av = A.view({"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dt]).float().double()[:, :m]
    if sc is not None:
        Av = Av * sc.double()[:, None]
    B = torch.zeros(r, (m + 3) // 4 * 4, device="cuda")
    B[:, :m] = torch.randn(r, m, generator=gen, device="cuda")
    for target in (None, B):
        kw = dict(r_max=r, batched=(2, k, k)) if target is not None else dict(self_target=True)
        s = gpu.Selector(A, m, k_max=k, scales=sc, **kw)
        s.set_target(target)
        W = torch.zeros(k, n, device="cuda")
        s.set_embedding(W)
        for pd in (1, 2):
            s.tuning(stream_pd=pd)
            W.zero_()
            assert s.select(k)[2] == k
            Q = torch.from_numpy(s.read(gpu.STATE_Q, m * k, np.float64).reshape(k, m)).cuda()
            assert torch.max((W.double() - Q @ Av.T).abs() / Av.norm(dim=1)[None, :]) <= 1e-5
        if target is not None:
            ib, im, om, nm, _ = s.select_batched(np.array([0, 140, n]), k, k)
            assert nm == k and np.all(ib[0] < 140) and np.all(ib[1] >= 140)
            best = ((Av @ B[:, :m].double().T) ** 2).sum(1) / (Av * Av).sum(1)
            for b, (lo, hi) in enumerate(((0, 140), (140, n))):
                assert best[ib[b][0]] >= (1 - 1e-5) * best[lo:hi].max()
        s.close()
