"""Reductions of a training step at the edges of their workgroups (64 rows by
16 columns for the bias gradient, 64 tiles for the loss), against float64 sums
of the network's own float32 outputs.  A float32 sum of B terms is off by at
most (B + 8) 2^-24 of the terms' magnitudes; the loss is a float64 sum rounded
once."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_out,B", [(1, 32), (15, 64), (16, 96), (17, 32), (33, 2080), (800, 1024), (3200, 160)])
def test_output_bias_gradient_and_loss(n_out, B):
    from paper_2602_06688_amd import pwfs as P
    rng = np.random.default_rng(n_out + B)
    mlp = P.MLP([32, n_out], max_batch=B, precision=P.BF16)
    mlp.set_params(torch.from_numpy((rng.standard_normal(33 * n_out) * 0.3).astype(np.float32)).cuda())
    x = torch.from_numpy(rng.standard_normal((B, 32)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.standard_normal((B, n_out)).astype(np.float32)).cuda()
    print(f"[gpu] train reductions n_out={n_out} B={B}", flush=True)
    y = mlp.forward(x)
    g = torch.zeros(mlp.n_params, dtype=torch.float32, device="cuda")
    loss = mlp.grad(x, t, grads=g)
    torch.cuda.synchronize()
    d = (y - t).double().cpu().numpy()
    dy = 2.0 * d / (B * n_out)
    gb = g.cpu().numpy()[-n_out:].astype(np.float64)
    assert (np.abs(gb - dy.sum(0)) <= (B + 8) * 2.0 ** -24 * np.abs(dy).sum(0)).all()
    assert abs(float(loss.item()) / (d * d).mean() - 1.0) <= 1e-6


@pytest.mark.parametrize("prec", ["BF16", "BF16X3"])
@pytest.mark.parametrize("M,N,K", [(1, 1024, 32), (63, 1024, 96), (65, 1000, 64), (200, 1023, 192), (4032, 1024, 416),
                                   (5, 9, 1), (130, 70, 33)])
def test_small_tiles_give_the_bits_of_the_large_ones(prec, M, N, K):
    """Rows of a product computed alone (64 x 64 tiles) and inside one of 8192
    rows (the tiles of products that fill the chip): every element adds the same
    matrix products in the same order."""
    from paper_2602_06688_amd import pwfs as P
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(8192, K, device="cuda", generator=g)
    B = torch.randn(N, K, device="cuda", generator=g)
    print(f"[gpu] gemm {prec} {M} of 8192 x {N} x {K}", flush=True)
    whole = P.gemm(A, B, precision=getattr(P, prec))
    part = P.gemm(A[:M].contiguous(), B, precision=getattr(P, prec))
    torch.cuda.synchronize()
    assert torch.equal(part, whole[:M])
