"""The streaming pass holds its results in LDS and writes them at the end of a
team's columns, or earlier when the buffer is full: the same bits whether a
team's range fits the buffer (large units) or overflows it (many small units),
for the scores, the embedding and the picks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,self_target,dt", [
    (40, 500_001, False, "f32"),   # 6 units held per team
    (40, 500_001, True, "f32"),
    (600, 300_000, False, "bf16"),  # 12
    (600, 300_000, True, "bf16"),
    (300, 120_000, True, "fp8"),
])
def test_held_results_do_not_depend_on_the_units(gpu, m, n, self_target, dt):
    import torch
    k, r = 6, 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n)
    lda = (m + 255) // 256 * 256
    A32 = torch.zeros(n, lda, device="cuda")
    A32[:, :m] = torch.randn(n, 12, generator=gen, device="cuda") @ torch.randn(12, m, generator=gen, device="cuda")
    A32[:, :m] += 0.1 * torch.randn(n, m, generator=gen, device="cuda")
    A, sc = (A32, None) if dt == "f32" else gpu.quantize_tensor(A32, m, dt)
    s = gpu.Selector(A, m, k_max=k, r_max=r, self_target=self_target, scales=sc)
    W = torch.empty(k, n, device="cuda")
    s.set_embedding(W)
    B = None
    if not self_target:
        B = torch.zeros(r, (m + 63) // 64 * 64, device="cuda")
        B[:, :m] = torch.randn(r, m, generator=gen, device="cuda")
    s.set_target(B)
    got = []
    for upw in (1, 64):
        s.tuning(stream_upw=upw)
        W.fill_(float("nan"))
        idx, obj, ns, _ = s.select(k)
        assert ns == k
        got.append((idx, s.read(gpu.STATE_F, n, np.float64), s.read(gpu.STATE_G, n, np.float64),
                    W.cpu().numpy(), obj))
    for a, b in zip(got[0][:4], got[1][:4]):
        np.testing.assert_array_equal(a, b)
    assert np.all(np.isfinite(got[0][3]))
    assert np.max(np.abs(got[0][4] - got[1][4])) <= 1e-12 * got[0][4][0]
    s.close()
