"""Launches that carry several small steps: the row selection (count, compaction, copy, clearing),
the row kernel that counts the batch itself, and the kernel that finishes dX and sums the loss.
Compared with plain torch in 64 bits at the sizes where a rule changes over."""
import math

import pytest
import torch

from test_guarded_product_gpu import reference

pytestmark = pytest.mark.gpu
TOL = {torch.float32: 2e-6, torch.bfloat16: 8e-3}   # as in the product tests


def make(BT, H, V, dtype, ignore, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn(BT, H, device="cuda", generator=g).to(dtype)
    W = (torch.randn(V, H, device="cuda", generator=g) * 0.05).to(dtype)
    t = torch.randint(0, V, (BT,), device="cuda", generator=g)
    if ignore == "front":
        t[:BT // 2] = -100
    elif ignore == "row 0":
        t[0] = -100
    elif ignore == "all but one":
        t[torch.arange(BT, device="cuda") != BT // 2] = -100
    elif ignore == "all":
        t[:] = -100
    elif ignore == "scattered":
        t[torch.rand(BT, device="cuda", generator=g) < 0.3] = -100
    return X, W, t


def check(got, X, W, t, dtype):
    loss, dX, dW = got
    torch.cuda.synchronize()
    rl, rX, rW = reference(X.float(), W.float(), t)
    tol = TOL[dtype]
    if dtype == torch.float32:
        # a sum over K is rounded 6 K / 16 times (six plane products per 16 K), 2^-24 of the running
        # sum each, random signs: past K = 3000 that is more than the 2e-6 stated for short sums
        tol = max(tol, 2.0 ** -24 * math.sqrt(6 * max(X.shape[0], *W.shape) / 16))
    assert abs(float(loss) - rl) <= max(2e-6, tol / 4) * max(abs(rl), 1e-30)
    for name, a, b in (("dX", dX, rX), ("dW", dW, rW)):
        err = float((a.double().cpu() - b).norm() / b.norm().clamp(min=1e-30))
        assert err <= tol, (name, err)
    assert (dX[t == -100] == 0).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ignore", ["none", "front", "row 0", "all but one", "all", "scattered"])
@pytest.mark.parametrize("compaction", [True, False])
@pytest.mark.parametrize("BT", [1, 5, 259])
def test_row_selection(dtype, ignore, compaction, BT):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, 64, 300, dtype, ignore, BT)
    check(flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(row_compaction=compaction)), X, W, t, dtype)


@pytest.mark.parametrize("BT", [1536, 1537, 4097, 32768, 32769])   # counted by the row kernel; 5 rows per workgroup; both sides of the one-launch selection
@pytest.mark.parametrize("compaction", [True, False])
def test_rules_change_over_with_the_row_count(BT, compaction):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, 32, 70, torch.float32, "scattered", BT)
    check(flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(row_compaction=compaction)), X, W, t, torch.float32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ignore", ["none", "front", "all but one", "all", "scattered"])
def test_selection_over_several_chunks(dtype, ignore):
    # 5 launches of 256 rows at most; the valid rows are dealt to the last ones
    import paper_2410_10989_amd as flce
    X, W, t = make(1200, 64, 320, dtype, ignore, 5)
    o = flce.flce_options(logits_budget_bytes=256 * 320 * X.element_size(), row_compaction=True)
    check(flce.flce_fwd_bwd_opt(X, W, t, o), X, W, t, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("H,V", [(64, 320), (256, 9000), (66, 2600)])   # dX whole, cut along K, cut with odd rows
@pytest.mark.parametrize("flags", [0, 1, 2])
def test_heads_and_skipped_gradients(dtype, H, V, flags):
    import paper_2410_10989_amd as flce
    X, W, t = make(150, H, V, dtype, "scattered", 9)
    _, W2, t2 = make(150, H, V, dtype, "front", 10)
    loss, heads, dX, dWs = flce.flce_multihead_fwd_bwd(X, [W, W2], [t, t2], [1.0, 0.5], flags=flags)
    torch.cuda.synchronize()
    r1, r2 = reference(X.float(), W.float(), t), reference(X.float(), W2.float(), t2)
    tol = TOL[dtype]
    assert abs(float(loss) - (r1[0] + 0.5 * r2[0])) <= max(2e-6, tol / 4) * abs(r1[0])
    assert abs(float(heads[1]) - r2[0]) <= max(2e-6, tol / 4) * abs(r2[0])
    want = r1[1] + 0.5 * r2[1]
    if not flags & flce.SKIP_DX:
        assert float((dX.double().cpu() - want).norm() / want.norm()) <= tol
    if not flags & flce.SKIP_DW:
        assert float((dWs[1].double().cpu() - 0.5 * r2[2]).norm() / (0.5 * r2[2]).norm()) <= tol


@pytest.mark.parametrize("BT", [1, 1536, 1537])
@pytest.mark.parametrize("noalloc", [True, False])
@pytest.mark.parametrize("ignore", ["row 0", "all", "scattered"])
def test_cross_entropy_counts_its_rows(BT, noalloc, ignore):
    import paper_2410_10989_amd as flce
    Z, _, t = make(BT, 333, 333, torch.float32, ignore, BT + 1)
    z = Z.double()
    ok = (t != -100).double()[:, None]
    n = max(1.0, float(ok.sum()))
    lse = torch.logsumexp(z, 1, keepdim=True)
    at = t.clamp(min=0)[:, None]
    want = torch.exp(z - lse).scatter_add(1, at, torch.full_like(lse, -1.0)) * ok / n
    rl = float(((lse - z.gather(1, at)) * ok).sum()) / n
    loss = torch.empty((), device="cuda")
    flce.flce_cross_entropy_inplace(Z, t, -100, loss=loss, noalloc=noalloc)
    torch.cuda.synchronize()
    assert abs(float(loss) - rl) <= 2e-6 * max(1.0, abs(rl))
    assert float((Z.double() - want).norm()) <= 2e-6 * max(float(want.norm()), 1e-30)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("BT,H,V,budget_rows,offset", [
    (70, 64, 300, 0, 0),       # normalised by the selection; dX finished beside dW, losses summed by the norm's backward
    (70, 64, 300, 0, 1),       # gamma not 16-byte aligned: the scalar forms
    (700, 264, 900, 256, 0),   # three chunks: the first starts the dgamma sums, the others add
    (33000, 32, 70, 0, 0),     # past the one-launch selection
    (40, 66, 200, 0, 0),       # rows that are not whole vectors (no compaction in bf16)
])
@pytest.mark.parametrize("flags", [0, 1, 2])
def test_rmsnorm_in_the_fused_launches(dtype, BT, H, V, budget_rows, offset, flags):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, "scattered", BT + H)
    g = torch.Generator(device="cuda").manual_seed(4)
    gamma = (1 + 0.1 * torch.randn(H + offset, device="cuda", generator=g)).to(dtype)[offset:]
    old = flce.flce_get_logits_budget_bytes()
    try:
        flce.flce_set_logits_budget_bytes(budget_rows * ((V + 63) // 64 * 64) * X.element_size())
        loss, dh, dgamma, dW = flce.flce_rmsnorm_fwd_bwd(X, gamma, 1e-6, W, t, flags=flags)
        torch.cuda.synchronize()
    finally:
        flce.flce_set_logits_budget_bytes(old)
    x, gm = X.double().cpu(), gamma.double().cpu()
    rms = torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6)
    xhat = x / rms
    y = (xhat * gm).to(dtype)          # what the products see
    rl, dY, rW = reference(y.float(), W.float(), t)
    a = dY * gm
    want_h = (a - (xhat * a).mean(1, keepdim=True) * xhat) / rms
    want_g = (dY * xhat).sum(0)
    tol = TOL[dtype] if dtype == torch.bfloat16 else max(TOL[dtype], 2.0 ** -24 * math.sqrt(6 * max(BT, H, V) / 16))
    assert abs(float(loss) - rl) <= max(2e-6, tol / 4) * abs(rl)
    if not flags & flce.SKIP_DX:
        assert float((dh.double().cpu() - want_h).norm() / want_h.norm()) <= tol
        assert float((dgamma.double().cpu() - want_g).norm() / want_g.norm()) <= 4 * tol   # BT signed terms per column
    if not flags & flce.SKIP_DW:
        assert float((dW.double().cpu() - rW).norm() / rW.norm()) <= tol


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_lent_workspace_below_the_fast_plan(dtype):
    # a buffer lent to the device that lacks room for the finer K ranges of dX still serves: the call
    # takes the plan of the large tiles (the room a caller may have set aside for that)
    import paper_2410_10989_amd as flce
    BT, H, V = 600, 256, 16384
    X, W, t = make(BT, H, V, dtype, "scattered", 12)
    code = flce.FLCE_F32 if dtype == torch.float32 else flce.FLCE_BF16
    need = flce.flce_workspace_bytes(BT, H, V, code)
    buf = torch.full((need - 256,), 255, dtype=torch.uint8, device="cuda")
    off = -buf.data_ptr() % 256
    try:
        flce.flce_set_workspace(buf[off:])
        check(flce.flce_fwd_bwd(X, W, t), X, W, t, dtype)
    finally:
        flce.flce_set_workspace(None)


@pytest.mark.parametrize("BT,H,V,compacted", [
    (600, 256, 16384, True),     # dX cut into more K ranges than the buffer has room for
    (1500, 72, 700, False),      # H % 64 != 0, dX not cut: no room for the index maps either
    (1911, 968, 16916, False),   # both
])
@pytest.mark.parametrize("how", ["options", "lent", "rmsnorm"])
def test_workspace_without_the_fast_plan(BT, H, V, compacted, how):
    # a buffer with room for the large tiles' K ranges only (what an explicit budget reports) and, with
    # H % 64 != 0, without row compaction, serves however it is passed; 256 bytes less are refused
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, torch.bfloat16, "scattered", 31)
    auto = max(1 << 30, 4096 * ((V + 63) // 64 * 64) * 2)
    o = flce.flce_options(logits_budget_bytes=auto, row_compaction=compacted)
    need = flce.flce_workspace_bytes_opt(BT, H, V, flce.FLCE_BF16, o)
    assert need < flce.flce_workspace_bytes(BT, H, V, flce.FLCE_BF16)
    if how == "rmsnorm":   # rstd and the 512 partial sums of dgamma
        need += (4 * BT + 255) // 256 * 256 + 512 * H * 4
    buf = torch.full((need + 256,), 255, dtype=torch.uint8, device="cuda")
    at = -buf.data_ptr() % 256

    def call(nbytes):
        ws = buf[at:at + nbytes]
        if how == "options":
            return flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(workspace=ws))
        try:
            flce.flce_set_workspace(ws)
            if how == "lent":
                return flce.flce_fwd_bwd(X, W, t)
            ones = torch.ones(H, dtype=torch.bfloat16, device="cuda")
            loss, dh, _, dW = flce.flce_rmsnorm_fwd_bwd(X, ones, 1e-6, W, t)
            return loss, dh, dW
        finally:
            torch.cuda.synchronize()
            flce.flce_set_workspace(None)

    got = call(need)
    if how == "rmsnorm":
        x = X.double()
        y = (x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6)).to(torch.bfloat16)
        rl, _, rW = reference(y.float(), W.float(), t)
        assert abs(float(got[0]) - rl) <= 2e-3 * rl
        assert float((got[2].double().cpu() - rW).norm() / rW.norm()) <= TOL[torch.bfloat16]
    else:
        check(got, X, W, t, torch.bfloat16)
    with pytest.raises(flce.FlceError):
        call(need - 256)


@pytest.mark.parametrize("share", [0.0, 0.5, 1.0])   # of the room between the bounded plan's and the full one's
def test_product_that_streams_w_in_any_room(share):
    # operands beyond the memory-side cache: dX in up to two workgroups per CU, fewer ranges in less room
    import paper_2410_10989_amd as flce
    BT, H, V = 24, 3584, 40003
    X, W, t = make(BT, H, V, torch.bfloat16, "scattered", 7)
    bounded = flce.flce_workspace_bytes_opt(BT, H, V, flce.FLCE_BF16, flce.flce_options(logits_budget_bytes=1 << 30))
    full = flce.flce_workspace_bytes(BT, H, V, flce.FLCE_BF16)
    assert bounded < full
    buf = torch.full((full + 256,), 255, dtype=torch.uint8, device="cuda")
    at = -buf.data_ptr() % 256
    ws = buf[at:at + bounded + int((full - bounded) * share)]
    check(flce.flce_fwd_bwd_opt(X, W, t, flce.flce_options(workspace=ws)), X, W, t, torch.bfloat16)


@pytest.mark.parametrize("BT,H,V,ranges", [
    (257, 512, 180001, 64),    # 2 x 2 large tiles, as many ranges as there are
    (700, 512, 128256, 42),    # 3 x 2 tiles: 252 workgroups
    (1024, 512, 128256, 32),
])
@pytest.mark.parametrize("ignored", [0, 0.5])
def test_streaming_product_in_one_round_of_large_tiles(BT, H, V, ranges, ignored):
    # with rows ignored the ranges stay (one round holds them all), over fewer tiles.  Against plain torch in 64
    # bits; bf16 storage of logits, gradients and results: TOL, a lost range would be 1 / 64 of dX's norm or more.
    import paper_2410_10989_amd as flce
    assert flce.flce_dx_k_ranges(BT, H, V, flce.FLCE_BF16) == ranges
    g = torch.Generator(device="cuda").manual_seed(BT)
    X = torch.randn(BT, H, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, H, device="cuda", generator=g) * 0.02).bfloat16()
    t = torch.randint(0, V, (BT,), device="cuda", generator=g)
    t[torch.rand(BT, device="cuda", generator=g) < ignored] = -100
    _, dX, _ = flce.flce_fwd_bwd(X, W, t, flags=flce.SKIP_DW)
    ok = t != -100
    x, w = X[ok].double(), W.double()
    G = torch.softmax(x @ w.T, 1)
    G[torch.arange(len(x), device="cuda"), t[ok]] -= 1.0
    want = (G / len(x)) @ w
    err = float((dX[ok].double() - want).norm() / want.norm())
    print(f"  {BT} x {H} x {V}, {ignored} ignored: {err:.1e}", flush=True)
    assert err <= TOL[torch.bfloat16]
    assert (dX[~ok] == 0).all()


@pytest.mark.parametrize("BT", [8192, 8193])   # 32 chunks of 256 rows selected by one launch each; 33 found with the cursor
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_selection_changes_over_with_the_chunk_count(BT, dtype):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, 32, 70, dtype, "scattered", BT)
    o = flce.flce_options(logits_budget_bytes=256 * 128 * X.element_size(), row_compaction=True)
    check(flce.flce_fwd_bwd_opt(X, W, t, o), X, W, t, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ignore", ["scattered", "front", "all"])
@pytest.mark.parametrize("BT,H,V", [
    (3, 8, 300),         # the smallest: one tile row with three rows
    (130, 72, 1000),     # two tile rows, a K tail (bf16)
    (256, 128, 2000),    # one chunk of at most 256 rows: rotated K loop (bf16)
    (257, 1024, 700),    # long K loops in 16 tiles and more
    (257, 1032, 700),
    (30, 1024, 384),     # fewer than 16 tiles, the longest K loop that still has its rows picked; 1032: no longer
    (30, 1032, 384),
    (2048, 64, 600),     # the longest batch; 2049: a launch of its own
    (2049, 64, 600),
])
def test_rows_picked_by_the_logits_launch(dtype, ignore, BT, H, V):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, ignore, BT + H)
    X[t == -100] = float("inf")   # rows without a target are never read into a sum
    got = flce.flce_fwd_bwd(X, W, t)
    X[t == -100] = 0
    check(got, X, W, t, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("BT,H,V,picked", [(257, 1032, 700, True), (30, 1024, 384, True), (30, 1032, 384, False),
                                           (2048, 64, 600, True), (2049, 64, 600, False)])
def test_which_batches_have_their_rows_picked(dtype, BT, H, V, picked):
    # the launch of its own is the only one of these calls that is neither a product nor the cross entropy
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, "scattered", 4)
    flce.flce_fwd_bwd(X, W, t)
    flce.flce_timing_collect()
    flce.flce_timing_enable(True)
    try:
        flce.flce_fwd_bwd(X, W, t)
    finally:
        flce.flce_timing_enable(False)
    assert flce.flce_timing_collect()["other"][1] == (0 if picked else 1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_picked_rows_are_gathered_for_dw_only(dtype):
    import paper_2410_10989_amd as flce
    X, W, t = make(300, 64, 700, dtype, "none", 6)
    ws = torch.zeros(flce.flce_workspace_bytes(300, 64, 700, flce.FLCE_F32 if dtype == torch.float32 else flce.FLCE_BF16) + 256,
                     dtype=torch.uint8, device="cuda")
    row = X[200].cpu().view(torch.uint8).numpy().tobytes()
    flce.flce_set_workspace(ws[-ws.data_ptr() % 256:])
    try:
        for flags in (flce.SKIP_DW, 0):
            flce.flce_fwd_bwd(X, W, t, flags=flags)
            torch.cuda.synchronize()
            assert (row in ws.cpu().numpy().tobytes()) == (flags == 0)
    finally:
        flce.flce_set_workspace(None)


def test_out_of_range_operands_of_picked_rows():
    # fp32: an infinity in a picked row sends its tile to the fp32 instructions, which look the rows up again
    import paper_2410_10989_amd as flce
    X, W, t = make(300, 64, 700, torch.float32, "scattered", 9)
    row = int((t != -100).nonzero()[100])
    X[row, 5] = 1e32
    W[:, 5] = 0
    loss, dX, dW = flce.flce_fwd_bwd(X, W, t)
    X2 = X.clone()
    X2[row, 5] = 0   # times zero weights: the same logits; dW's column 5 apart
    rl, rX, rW = reference(X2, W, t)
    assert abs(float(loss) - rl) <= 2e-6 * abs(rl)
    keep = torch.arange(64) != 5
    for a, b in ((dX.cpu()[:, keep], rX[:, keep]), (dW.cpu()[:, keep], rW[:, keep])):
        assert float((a.double() - b).norm() / b.norm()) <= TOL[torch.float32]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("BT,H,V", [
    (1, 8, 130),        # one row, a tile of 8 columns (fp32: 64-tiles, bf16: 128-tiles)
    (64, 64, 127),      # whole 64-tiles, ragged vocabulary
    (129, 136, 300),    # one row and one 8-column strip past a 128-tile
    (300, 264, 700),    # dX in K ranges (fp32), not (bf16)
    (200, 72, 3000),    # dX in K ranges
    (1500, 200, 1100),
])
@pytest.mark.parametrize("heads", [1, 2])
@pytest.mark.parametrize("skip_dw", [False, True])
def test_both_gradients_in_one_launch(dtype, BT, H, V, heads, skip_dw):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, "scattered" if BT > 1 else "none", BT + V)
    Ws, ts = [W], [t]
    if heads == 2:
        Ws.append((W.flip(0) * 0.5).contiguous())
        ts.append(torch.where(t == -100, t, (t * 7 + 1) % V))
    weights = [1.0, 0.7][:heads]
    dX = torch.full_like(X, float("nan"))
    loss, _, dX, dWs = flce.flce_multihead_fwd_bwd(X, Ws, ts, weights, dX=dX, flags=flce.SKIP_DW if skip_dw else 0)
    torch.cuda.synchronize()
    refs = [reference(X.float(), w.float(), u) for w, u in zip(Ws, ts)]
    tol = TOL[dtype] if dtype == torch.bfloat16 else max(TOL[dtype], 2.0 ** -24 * math.sqrt(6 * max(BT, H, V) / 16))
    want = sum(c * r[0] for c, r in zip(weights, refs))
    assert abs(float(loss) - want) <= max(2e-6, tol / 4) * max(abs(want), 1e-30)
    rX = sum(c * r[1] for c, r in zip(weights, refs))
    assert float((dX.double().cpu() - rX).norm() / rX.norm()) <= tol
    assert (dX[t == -100] == 0).all()
    for c, r, d in zip(weights, refs, dWs or []):
        assert float((d.double().cpu() - c * r[2]).norm() / (c * r[2]).norm()) <= tol


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("BT,H,V", [(60, 64, 300), (200, 72, 3000)])   # dX uncut, dX in K ranges
def test_both_gradients_in_one_launch_behind_rmsnorm(dtype, BT, H, V):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, "scattered", 5)
    ones = torch.ones(H, dtype=dtype, device="cuda")
    loss, dh, dgamma, dW = flce.flce_rmsnorm_fwd_bwd(X, ones, 1e-6, W, t)
    x = X.double().cpu()
    rms = torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6)
    xhat = x / rms
    rl, rY, rW = reference(xhat, W.float(), t)
    rh = (rY - (xhat * rY).mean(1, keepdim=True) * xhat) / rms
    # bf16: the normalised rows are rounded too, one rounding of 2^-9 more than in the plain call
    tol = 2 * TOL[dtype] if dtype == torch.bfloat16 else max(4e-6, 2.0 ** -23 * math.sqrt(6 * V / 16))
    assert abs(float(loss) - rl) <= tol * rl
    for a, b in ((dh, rh), (dgamma, (rY * xhat).sum(0)), (dW, rW)):
        assert float((a.double().cpu() - b).norm() / b.norm()) <= tol


@pytest.mark.parametrize("dtype,BT,H,V,skip_dw,dx,dw", [
    (torch.float32, 256, 512, 4096, False, 2, 1),   # both gradients in a launch, one that adds dX's K ranges up
    (torch.bfloat16, 18, 960, 384, False, 1, 1),    # one launch in all
    (torch.bfloat16, 44, 368, 110, True, 1, 0),
])
def test_timing_of_launches_that_do_several_things(dtype, BT, H, V, skip_dw, dx, dw):
    import paper_2410_10989_amd as flce
    X, W, t = make(BT, H, V, dtype, "scattered", 3)
    call = lambda: flce.flce_fwd_bwd(X, W, t, flags=flce.SKIP_DW if skip_dw else 0)
    call()
    flce.flce_timing_collect()
    flce.flce_timing_enable(True)
    try:
        call()
    finally:
        flce.flce_timing_enable(False)
    kinds = flce.flce_timing_collect()
    # the rows are selected in the logits launch: nothing is left for "other"
    assert {k: n for k, (_, n) in kinds.items()} == {"logits_gemm": 1, "ce_rows": 1, "dx_gemm": dx, "dw_gemm": dw, "other": 0}
    assert all((ms > 0) == (n > 0) for ms, n in kinds.values())
    if dw:   # half of the launch each; dX's share has the rest of its own time on top
        assert kinds["dx_gemm"][0] == kinds["dw_gemm"][0] if dx == 1 else kinds["dx_gemm"][0] > kinds["dw_gemm"][0]
