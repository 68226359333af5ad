"""The tuned bf16 product kernel at the edges of its two tile sizes and of a K step, through the
entry point, against plain torch in 64 bits on the same bf16 inputs."""
import pytest
import torch

from test_guarded_product_gpu import inputs, reference

pytestmark = pytest.mark.gpu

# What bf16 storage costs: logits |z| of about 1 stored to 2^-9 relative (their exponentials move by
# as much), the logit gradients and the results rounded to 2^-9 each: at most about 4 * 2^-9 = 8e-3
# of a result's norm if all of it lined up, 2e-3 .. 3e-3 measured.  A lost K piece of 8, a row or
# column taken from a neighbour, or a K range left out changes the result by 3e-2 or more.
TOL = 8e-3


def check(BT, H, V, compaction=True):
    import paper_2410_10989_amd as flce
    X, W, t = inputs(BT, H, V, 3 * BT + V)
    X, W = X.bfloat16(), W.bfloat16()
    o = flce.flce_options(row_compaction=compaction)
    loss, dX, dW = flce.flce_fwd_bwd_opt(X, W, t, o)
    torch.cuda.synchronize()
    rl, rX, rW = reference(X.float(), W.float(), t)
    print(f"  {BT} x {H} x {V} compaction {compaction}: loss {abs(float(loss) / rl - 1):.1e}", end="")
    assert abs(float(loss) - rl) <= 2e-3 * abs(rl)
    for name, got, ref in (("dX", dX, rX), ("dW", dW, rW)):
        err = float((got.double().cpu() - ref).norm() / ref.norm())
        print(f" {name} {err:.1e}", end="", flush=True)
        assert err <= TOL, (name, err)
    print(flush=True)


@pytest.mark.parametrize("BT,H,V", [
    (128, 64, 128),       # one 128 x 128 tile in the logits and dW products, one K step
    (129, 128, 130),      # one row and column past a tile
    (127, 72, 257),       # H: one K step and a piece of 8
    (1, 8, 128),          # a K step with a single piece; one row
    (300, 120, 4097),     # H: a K step that lacks its last piece; K ranges of dX with a ragged end
    (1024, 512, 8192),    # 128-tiles in all three products, 8 K ranges
    (2000, 1000, 3001),   # H = 15 whole K steps and 40: tail in the last of many steps
    (2047, 1000, 50257),  # 256-tiles with a K tail, dX in 8 K ranges that fill one round
    (4500, 200, 16384),   # tall: 256-tiles with few K steps
])
@pytest.mark.parametrize("compaction", [True, False])
def test_tile_edges_and_k_tails(BT, H, V, compaction):
    check(BT, H, V, compaction)


def test_k_ranges_of_both_tile_sizes():
    # (which tile size the rule picks at these sizes is checked on the CPU)
    import paper_2410_10989_amd as flce
    assert flce.flce_dx_k_ranges(1024, 512, 8192, flce.FLCE_BF16) == 8       # 8 x 4 tiles of 128 x 128
    assert flce.flce_dx_k_ranges(2047, 1000, 50257, flce.FLCE_BF16) == 8     # 8 x 4 tiles of 256 x 256
    assert flce.flce_dx_k_ranges(4096, 4096, 32000, flce.FLCE_BF16) == 1
