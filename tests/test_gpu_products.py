"""Products on either side of the line between 64 x 64 and 128 x 128 tiles, with
remainders in every size: the rows computed alone and inside a product of 8192
rows have the same bits, and both are within the operands' rounding of the
float64 product.

An operand is held as bfloat16 (relative error 2^-8) or as two of them (2^-16, the
product of the two low parts, at most 2^-16, left out); K float32 additions err by
at most K 2^-24 of the terms' magnitudes."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

REL = {"BF16": 2 * 2.0 ** -8 + 2.0 ** -16, "BF16X3": 3 * 2.0 ** -16}


@pytest.mark.parametrize("prec", ["BF16", "BF16X3"])
@pytest.mark.parametrize("M,N,K", [
    (5, 1024, 1), (130, 1030, 33), (65, 1023, 500), (1, 1025, 95),
    (1000, 1729, 40),           # 112 tiles
    (2431, 1217, 70),           # 190: below both lines
    (2432, 1280, 97),           # 190, whole tiles
    (2559, 1920, 33),           # 300
    (2560, 2047, 65),           # 320
    (2433, 2049, 31),           # 340: above both
])
def test_remainders_on_both_sides_of_the_tile_rule(prec, M, N, K):
    from paper_2602_06688_amd import pwfs as P
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(8192, K, device="cuda", generator=g)
    B = torch.randn(N, K, device="cuda", generator=g)
    print(f"[gpu] products {prec} {M} of 8192 x {N} x {K}", flush=True)
    whole = P.gemm(A, B, precision=getattr(P, prec))
    part = P.gemm(A[:M].contiguous(), B, precision=getattr(P, prec))
    torch.cuda.synchronize()
    assert torch.equal(part, whole[:M])
    want = A[:M].double() @ B.double().T
    bound = (REL[prec] + (K + 8) * 2.0 ** -24) * (A[:M].abs().double() @ B.abs().double().T)
    assert bool(((part.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("prec", ["BF16", "BF16X3"])
@pytest.mark.parametrize("hidden,batch", [(1030, 100), (1030, 2600), (1030, 8200), (1030, 16000), (2050, 16400)])
def test_rows_of_a_prediction_do_not_depend_on_its_batch(prec, hidden, batch):
    """Hidden layers of 9, 189, 585, 1125 and 2193 tiles (64 x 64, 128 x 128
    wave-specialised, 256-lane) and the output layers behind them give the rows of
    a batch of 70 their bits."""
    from paper_2602_06688_amd import pwfs as P
    g = torch.Generator(device="cuda").manual_seed(hidden + batch)
    mlp = P.MLP([33, hidden, 600], max_batch=32 * -(-batch // 32), precision=getattr(P, prec))
    mlp.set_params(torch.randn(mlp.n_params, device="cuda", generator=g) * 0.05)
    x = torch.randn(batch, 33, device="cuda", generator=g)
    print(f"[gpu] prediction {prec} hidden {hidden} batch {batch}", flush=True)
    few = mlp.forward(x[:70].contiguous()).clone()
    many = mlp.forward(x)
    torch.cuda.synchronize()
    assert torch.equal(few, many[:70]) and bool(torch.isfinite(many).all())
