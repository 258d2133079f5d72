"""The work predictor's gradient where its sums change shape: one chunk of
samples against several, a chunk's last part of 40 full or not, the most chunks
there are, and a forward pass whose last workgroup is full or not."""
import numpy as np
import pytest

from oracle import mlp_ref


@pytest.mark.gpu
@pytest.mark.parametrize("n", [40, 63, 64, 65, 79, 80, 81, 10239, 10240, 10401, 20500])
def test_gradient_at_chunk_edges(n):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    print(f"case mlp chunks n={n}", flush=True)
    rng = np.random.default_rng([37, n])
    theta = rng.normal(0, 0.25, mlp_ref.NPARAM).astype(np.float32)
    x = rng.normal(0, 1, (n, 4)).astype(np.float32)
    t = rng.normal(0, 1, n).astype(np.float32)
    P, X, T = (torch.from_numpy(a).cuda() for a in (theta, x, t))
    cache = torch.empty((n, 128), dtype=torch.float32, device="cuda")
    dz = torch.full((n * 129 + 64,), 7.5, dtype=torch.float32, device="cuda")  # guard words behind the scratch
    grad, grad2 = (torch.full((mlp_ref.NPARAM + 1,), 7.5, dtype=torch.float32, device="cuda") for _ in range(2))
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    y = bz.bz_mlp_forward(P, X, cache)
    bz.bz_mlp_backward(P, X, T, y, cache, dz, grad, loss)
    bz.bz_mlp_backward(P, X, T, y, cache, dz, grad2, None)
    assert torch.equal(grad, grad2), "a fixed order of sums"
    assert torch.all(dz[n * 129:] == 7.5) and grad[-1] == 7.5, "written past the end"
    y_ref, (_, h1, _, h2) = mlp_ref.forward(theta.astype(np.float64), x)
    # FP32 chains of at most 65 terms: 65 x 2^-24 = 4e-6 of the terms' sizes (below 20)
    assert np.abs(y.cpu().numpy() - y_ref).max() <= 1e-4
    assert np.abs(cache.cpu().numpy() - np.concatenate([h1, h2], axis=1)).max() <= 1e-4
    g_ref = mlp_ref.grad(theta.astype(np.float64), x, t)
    scale = np.abs(g_ref).max()
    # chains of 40 samples and of 64 rows, each product of relative error below 1e-5
    assert np.abs(grad[:-1].cpu().numpy() - g_ref).max() <= 1e-4 * scale + 1e-6
    assert abs(loss.item() - mlp_ref.loss(theta.astype(np.float64), x, t)) <= 1e-4 * max(1.0, loss.item())
