"""The block Jacobi's limit on sweeps: spectra that fall by seven to ten decades
(the entries of their small eigenvalues' block are within a few rounding errors
of the sweeps' zero) take 20 to 45 sweeps at these sizes, and none of them may
be given up.  Against the eigenvalues from numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [333, 500])
def test_steep_spectra_converge(gpu, l):
    m, n = l + 50, 2 * l
    rng = np.random.default_rng(l)
    A = np.zeros((n, (m + 63) // 64 * 64), np.float32)
    A[:, :m] = rng.standard_normal((n, m))
    s = gpu.Selector(torch.from_numpy(A).cuda(), m, k_max=l, self_target=True)
    s.set_target(None)
    W = torch.zeros(l, n, dtype=torch.float32, device="cuda")
    s.set_embedding(W)
    assert s.select(l)[2] == l
    V = np.linalg.qr(rng.standard_normal((n, l)))[0].T
    for decades in (7.0, 7.5, 8.0, 10.0):
        U = np.linalg.qr(rng.standard_normal((l, l)))[0]
        X = (U * 10.0 ** (-decades * np.arange(l) / l)) @ V
        W.copy_(torch.from_numpy(X))
        Wd = W.cpu().numpy().astype(np.float64)
        want = np.linalg.eigvalsh(Wd @ Wd.T)[::-1]
        _, sigma, _, _ = s.rank_k(l, l, want_u=False, want_v=False)
        # Jacobi in FP64: every sweep's l rotations per entry round by eps of the largest
        # eigenvalue, so eps l sweeps, here taken as eps l^2
        assert np.max(np.abs(np.asarray(sigma) ** 2 - np.maximum(want, 0.0))) <= 2.3e-16 * l * l * want[0]
    s.close()


@pytest.mark.parametrize("l", [1, 2])
def test_smallest_embeddings(gpu, l):
    m, n = 40, 300
    rng = np.random.default_rng(l)
    A = np.zeros((n, 64), np.float32)
    A[:, :m] = rng.standard_normal((n, m))
    s = gpu.Selector(torch.from_numpy(A).cuda(), m, k_max=l, self_target=True)
    s.set_target(None)
    W = torch.zeros(l, n, dtype=torch.float32, device="cuda")
    s.set_embedding(W)
    assert s.select(l)[2] == l
    Q = s.read(gpu.STATE_Q, m * l, np.float64).reshape(l, m)
    Uw, want, Vt = np.linalg.svd(W.cpu().numpy().astype(np.float64), full_matrices=False)
    U, sigma, V, _ = s.rank_k(l, l)
    np.testing.assert_allclose(sigma, want, rtol=1e-14)
    for j in range(l):
        u = Uw[:, j] @ Q
        sign = np.sign(u[np.argmax(np.abs(u))])
        assert np.max(np.abs(U[j].cpu().numpy() - sign * u)) <= 1e-13
        assert np.max(np.abs(V[j].cpu().numpy() - sign * Vt[j])) <= 1e-6
    s.close()
