"""The guarded product kernel (fp32 storage on split bf16 planes, any shape and alignment)
against plain torch in 64 bits: edges of its 64 and 128 tiles, K ranges, K tails, odd leading
dimensions, and operands the split cannot represent."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def reference(X, W, t):
    X, W = X.double().cpu(), W.double().cpu()
    t = t.cpu()
    ok = (t != -100).double()[:, None]
    n = max(1.0, float(ok.sum()))
    z = X @ W.T
    lse = torch.logsumexp(z, 1, keepdim=True)
    at = t.clamp(min=0)[:, None]
    loss = float(((lse - z.gather(1, at)) * ok).sum()) / n
    G = (torch.exp(z - lse).scatter_add(1, at, torch.full_like(lse, -1.0))) * ok / n
    return loss, G @ W, G.T @ X


def inputs(BT, H, V, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn(BT, H, device="cuda", generator=g)
    W = torch.randn(V, H, device="cuda", generator=g) * 0.05
    t = torch.randint(0, V, (BT,), device="cuda", generator=g)
    t[3::7] = -100
    return X, W, t


# One fp32 rounding per accumulation step: K/16 * 6 roundings of at most 2^-24 of the running sum,
# random signs: below 2^-24 * sqrt(6 K / 16) of the result; the operands' own rounding (logits,
# exponentials of them) adds a few 2^-24 |z|.  4e-7 .. 1e-6 for the sizes below, stated 2e-6: a lost
# plane product (2^-16 .. 2^-18 relative) would show as 4e-6 .. 1e-5.
@pytest.mark.parametrize("BT,H,V", [
    (64, 64, 64),        # one 64 x 64 tile
    (65, 33, 67),        # one row, column and K value past a tile and a K step; odd leading dimensions
    (127, 100, 1025),    # 64-tiles, dX cut into K ranges with a tail
    (129, 260, 4098),    # K ranges whose last one is ragged
    (1100, 516, 7001),   # 128-tiles in logits and dW, K ranges of 512 in dX, odd V
    (2049, 1030, 2111),  # 128-tiles everywhere, rows that are not 16-byte aligned
    (1, 7, 300),         # a single row
])
def test_fp32_products_keep_fp32_accuracy(BT, H, V):
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 7 * BT + V)
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    torch.cuda.synchronize()
    rl, rX, rW = reference(X, W, t)
    assert abs(float(loss) - rl) <= 2e-6 * abs(rl)
    for name, got, ref in (("dX", dX, rX), ("dW", dW, rW)):
        err = float((got.double().cpu() - ref).norm() / ref.norm())
        print(f"  {BT} x {H} x {V} {name}: {err:.2e}", flush=True)
        assert err <= 2e-6, (name, err)


@pytest.mark.parametrize("BT,H,V", [(100, 40, 300), (1100, 128, 7000)])   # 64 and 128 tiles
def test_operands_beyond_bf16_take_fp32_products(BT, H, V):
    # finite fp32 values that round to infinity in bf16 times tiny ones: ordinary logits; and a class
    # masked by a weight of -inf against positive activations: probability 0, everything else finite
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 11)
    t = torch.where(t == 5, torch.full_like(t, 6), t)
    X[:, 0] = 3.4e38
    W[:, 0] = torch.randn(V, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)) * 1e-38
    X[:, 1] = 1.0 + X[:, 1].abs()
    W[5, 1] = -float("inf")
    loss, _, dW = flce.flce_fwd_bwd(X, W, t, flags=flce.SKIP_DX)
    torch.cuda.synchronize()
    keep = torch.arange(V, device="cuda") != 5
    rl, _, rW = reference(X, W[keep], torch.where(t > 5, t - 1, t))
    assert abs(float(loss) - rl) <= 1e-5 * abs(rl)
    got = dW[keep].double().cpu()
    assert torch.isfinite(dW).all() and (dW[5] == 0).all()
    # column 0 of dW is sums of g * 3.4e38; compared on its own scale
    for sl in (slice(0, 1), slice(1, None)):
        assert float((got[:, sl] - rW[:, sl]).norm() / rW[:, sl].norm()) <= 1e-5


def test_nan_stays_where_plain_products_put_it():
    import paper_2410_10989_amd as flce
    X, W, t = inputs(300, 64, 500, 13)
    X[7, 3] = float("nan")
    t[7] = 1
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    torch.cuda.synchronize()
    assert torch.isnan(loss) and torch.isnan(dX[7]).all()
    ok = torch.arange(300, device="cuda") != 7
    n = int((t != -100).sum())
    _, rX, _ = reference(X[ok], W, t[ok])
    got = dX[ok].double().cpu() * n / (n - 1)     # the reference's mean is over one row less
    assert float((got - rX).norm() / rX.norm()) <= 2e-6


@pytest.mark.parametrize("BT,H,V", [(100, 40, 300), (1100, 128, 7000), (4096, 64, 16384)])   # 64, 128 and 256 tiles
@pytest.mark.parametrize("ex,ew", [(-124, 0), (0, -124), (-124, 124), (-100, 100)])
def test_small_operands_keep_fp32_accuracy(BT, H, V, ex, ew):
    # values near the smallest normal fp32, alone (dW = G^T X and dX = G W carry their relative error on)
    # and against partners that bring the logits back to order 1.  The scaling by powers of two is exact:
    # the same bound as for ordinary operands, plus the spacing of subnormal results (2^-149 per element;
    # up to 64 partial results of dX are rounded to it each, with random signs); 8 bits of a value
    # would show as 1e-3.
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 17)
    X, W = X * 2.0 ** ex, W * 2.0 ** ew
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    torch.cuda.synchronize()
    rl, rX, rW = reference(X, W, t)
    assert abs(float(loss) - rl) <= 2e-6 * abs(rl)
    for name, got, ref, parts in (("dX", dX, rX, 64), ("dW", dW, rW, 1)):
        err = float((got.double().cpu() - ref).norm())
        bound = 2e-6 * float(ref.norm()) + 2.0 ** -149 * math.sqrt(parts * ref.numel())
        print(f"  {BT} x {H} x {V} 2^{ex} 2^{ew} {name}: {err / float(ref.norm()):.2e} of {bound / float(ref.norm()):.2e}", flush=True)
        assert err <= bound, (name, err, bound)


def test_gradient_rows_of_improbable_classes():
    # classes of probability e^-83: their gradients, about 2^-127, enter dW on their own.  The logits'
    # own rounding moves the probabilities by |z| 2^-24 = 5e-6 and a few times that; 8 bits would be 1e-3.
    import paper_2410_10989_amd as flce
    X, W, t = inputs(100, 40, 300, 19)
    t = torch.where((t >= 100) & (t < 200), t - 100, t)
    X[:, 0] = 1.0
    W[100:200, 0] = -78.0
    loss, _, dW = flce.flce_fwd_bwd(X, W, t, flags=flce.SKIP_DX)
    torch.cuda.synchronize()
    _, _, rW = reference(X, W, t)
    err = float((dW[100:200].double().cpu() - rW[100:200]).norm() / rW[100:200].norm())
    print(f"  {err:.2e}", flush=True)
    assert err <= 5e-5


@pytest.mark.parametrize("BT,H,V", [(100, 40, 300), (1100, 128, 7000), (4096, 64, 16384), (513, 70, 300)])   # 64, 128, 256 tiles; odd rows
def test_a_nan_leaves_the_other_rows_their_bits(BT, H, V):
    # a NaN in one row of X makes that row's logits and dX, and all of dW, NaN; every other row of dX is
    # computed as it is without the NaN
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 23)
    t[7] = 1
    _, want, _ = flce.flce_fwd_bwd(X, W, t)
    X[7, 3] = float("nan")
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    torch.cuda.synchronize()
    assert torch.isnan(loss) and torch.isnan(dX[7]).all() and torch.isnan(dW).all()
    other = torch.arange(BT, device="cuda") != 7
    assert torch.equal(dX[other].view(torch.int32), want[other].view(torch.int32))


def test_sums_beyond_the_split_range():
    # operands within the range of the split whose sums are not (logits of 2^90): the largest logit wins,
    # probability 1, and an infinite one beside a NaN row
    import paper_2410_10989_amd as flce
    X, W, t = inputs(130, 33, 300, 29)
    X = X * 2.0 ** 60
    W = W * 2.0 ** 30
    z = X.double() @ W.double().T
    best = z.argmax(1)
    t = torch.where(t == -100, t, best)
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    torch.cuda.synchronize()
    assert float(loss) == 0.0 and (dX == 0).all() and (dW == 0).all()
    X[4, 5] = float("nan")
    X[9, 2] = float("inf")
    t[9] = -100
    loss, dX, dW = flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(row_compaction=False))
    torch.cuda.synchronize()
    other = torch.arange(130, device="cuda") != 4
    assert torch.isnan(loss) and torch.isnan(dX[4]).all() and (dX[other] == 0).all()


@pytest.mark.parametrize("BT,H,V", [(100, 40, 300), (1100, 128, 7000), (4096, 64, 16384)])   # 64, 128 and 256 tiles
def test_an_infinite_operand_is_computed_again_where_it_matters(BT, H, V):
    # an infinite activation in an ignored row (no compaction): 0 * inf = NaN in its column of dW, as in
    # plain products, and the rounding of ordinary sums everywhere else
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 37)
    t[9], X[9, 2] = -100, float("inf")
    loss, dX, dW = flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(row_compaction=False))
    torch.cuda.synchronize()
    ok = t != -100
    rl, rX, rW = reference(X[ok], W, t[ok])
    assert abs(float(loss) - rl) <= 2e-6 * abs(rl)
    assert torch.isnan(dW[:, 2]).all() and (dX[~ok] == 0).all()
    other = torch.arange(H) != 2
    assert float((dX[ok].double().cpu() - rX).norm() / rX.norm()) <= 2e-6
    assert float((dW.double().cpu() - rW)[:, other].norm() / rW[:, other].norm()) <= 2e-6
