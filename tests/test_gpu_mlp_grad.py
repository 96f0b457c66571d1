"""Network gradient over row counts at the edges of its 32-row wave tiles, of one
tile per workgroup (8,192 rows) and of one tile per wave (65,536 rows)."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def gradient_bound(p, X, t, mean, std):
    """Bound on |g_gpu - g| per parameter for FP32 arithmetic (u = 2^-24): the
    rounding of each dot product, the GELU and its derivative within 1e-6 of the
    erf formula's values (Abramowitz & Stegun 7.1.26, 1.5e-7, in FP32), errors
    carried through |GELU'| <= 1.13 and |GELU''| <= 0.8, and the sum over rows
    (chains of at most 64 + n / 256 additions)."""
    W1, b1, W2, b2, w3, b3 = mlp.unpack(p)
    y, (Z, z1, h1, z2, h2) = mlp.forward(p, X, mean, std)
    n, u, a = len(y), 2.0 ** -24, np.abs
    eg = 1e-6
    dz1e = 7 * u * (a(Z) @ a(W1).T + a(b1))
    h1e = 1.13 * dz1e + eg * (1 + a(z1))
    z2e = h1e @ a(W2).T + 66 * u * (a(h1) @ a(W2).T + a(b2))
    h2e = 1.13 * z2e + eg * (1 + a(z2))
    dy = 2 * a(y - t) / n
    dye = 2 / n * (h2e @ a(w3) + 66 * u * (a(h2) @ a(w3) + a(b3)) + 4 * u * (a(y) + a(t)))
    dz2 = dy[:, None] * a(w3) * 1.13
    dz2e = dye[:, None] * a(w3) * 1.13 + dy[:, None] * a(w3) * (eg + 0.8 * z2e) + 3 * u * dz2
    dh1, dh1e = dz2 @ a(W2), dz2e @ a(W2) + 66 * u * (dz2 @ a(W2))
    dz1 = dh1 * 1.13
    dz1g = dh1e * 1.13 + dh1 * (eg + 0.8 * dz1e) + 2 * u * dz1
    s = (64 + n / 256) * u
    out = np.zeros(mlp.NPARAM)
    out[mlp.OFF_W1:mlp.OFF_B1] = (dz1g.T @ a(Z) + dz1.T @ a(Z) * (s + 4 * u)).ravel()
    out[mlp.OFF_B1:mlp.OFF_W2] = dz1g.sum(0) + dz1.sum(0) * s
    out[mlp.OFF_W2:mlp.OFF_B2] = (dz2e.T @ a(h1) + dz2.T @ h1e + dz2.T @ a(h1) * s).ravel()
    out[mlp.OFF_B2:mlp.OFF_W3] = dz2e.sum(0) + dz2.sum(0) * s
    out[mlp.OFF_W3:mlp.OFF_B3] = dye @ a(h2) + dy @ h2e + dy @ a(h2) * s
    out[mlp.OFF_B3] = dye.sum() + dy.sum() * s
    return out + 1e-30


@pytest.mark.parametrize("n", [1, 31, 33, 8191, 8225, 65536 + 37])
def test_gradient_row_counts(n):
    import torch
    from paper_1608_01362_amd import warmstart as ws
    rng = np.random.default_rng(n)
    X = np.stack([rng.exponential(2, n), rng.exponential(1.5, n), rng.normal(2, 0.7, n)], axis=1).astype(np.float32)
    t = rng.normal(0, 1, n).astype(np.float32)
    net = ws.Network.create(3, [2.0, 1.5, 2.0], [2.0, 1.5, 0.7])
    # rows past n in the buffers: the gradient must not see them
    F = torch.full((n + 64, 3), float("nan"), device="cuda")
    T = torch.full((n + 64,), float("nan"), device="cuda")
    F[:n], T[:n] = torch.from_numpy(X), torch.from_numpy(t)
    norm = net.norm.double().cpu().numpy()
    p = net.weights.view(torch.bfloat16).double().cpu().numpy()
    args = (p, X.astype(np.float64), t.astype(np.float64), norm[:3], 1.0 / norm[3:])
    g, loss = net.grad(F[:n], T[:n])
    loss_ref, g_ref = mlp.loss_and_grad(*args)
    assert abs(float(loss.item()) - loss_ref) <= 1e-5 * loss_ref
    assert np.all(np.abs(g.double().cpu().numpy() - g_ref) <= gradient_bound(*args))
    g2, loss2 = net.grad(F[:n], T[:n])
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
