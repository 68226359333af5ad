"""The stand-alone cross entropy over rows that start at any address: head, vectors and tail of
the row kernel, each of its shapes, and targets in the head, at a vector's ends and in the tail."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-6), (torch.bfloat16, 4e-3)])   # fp32 exp and sums; one rounding to 2^-9
@pytest.mark.parametrize("V,ldz,offset", [
    (1, 1, 0), (5, 5, 1), (7, 9, 3),      # rows shorter than a vector: all head or tail
    (257, 257, 1),                        # 256-thread shape, a different head every row
    (24571, 24571, 5),                    # just under 48 KB of bf16, 96 KB of fp32
    (50257, 50257, 0),                    # 512-thread shape (bf16), 1024-thread shape (fp32)
    (57345, 57345, 3),                    # just past 112 KB of bf16
    (131073, 131077, 7),                  # past what the registers hold (fp32: and LDS)
    (204801, 204801, 1),                  # just past 400 KB of bf16: registers and LDS
    (262151, 262151, 2),                  # past both
])
def test_rows_at_any_address(dtype, tol, V, ldz, offset):
    import paper_2410_10989_amd as flce
    rows = 24
    g = torch.Generator(device="cuda").manual_seed(V + offset)
    flat = (torch.randn(offset + rows * ldz + 64, device="cuda", generator=g) * 2).to(dtype)
    Z = flat[offset:offset + rows * ldz].view(rows, ldz)[:, :V]
    t = torch.tensor([0, V - 1, V // 2, min(V - 1, 7), min(V - 1, 8), max(0, V - 9), max(0, V - 8), -100] * 3,
                     device="cuda")
    before = flat.clone()
    ref = Z.double()
    ok = t != -100
    lse = torch.logsumexp(ref, 1, keepdim=True)
    at = t.clamp(min=0)[:, None]
    want_loss = float(((lse - ref.gather(1, at))[:, 0] * ok).sum() / ok.sum())
    G = torch.exp(ref - lse).scatter_add(1, at, torch.full_like(lse, -1.0)) * ok[:, None] / ok.sum()
    loss = flce.flce_cross_entropy_inplace(Z, t, -100)
    torch.cuda.synchronize()
    assert abs(float(loss) - want_loss) <= 1e-6 * max(1.0, abs(want_loss))
    if V > 1:
        err = float((Z.double() - G).norm() / G.norm())
        print(f"  {V} {ldz} {offset} {dtype}: {err:.1e}", flush=True)
        assert err <= tol
        assert (Z[7] == 0).all()
    else:
        assert float(Z.double().abs().max()) <= 1e-6
    # nothing beside the rows is touched
    mask = torch.ones_like(flat, dtype=torch.bool)
    mask[offset:offset + rows * ldz].view(rows, ldz)[:, :V] = False
    assert torch.equal(flat[mask], before[mask])


@pytest.mark.parametrize("V", [64, 30000, 100003])   # one row length per shape of the kernel (bf16)
@pytest.mark.parametrize("rows", [1, 2, 511, 512, 513, 1024, 1025, 1536, 1537])   # both sides of what one launch serves
@pytest.mark.parametrize("noalloc", [False, True])
def test_loss_of_small_batches_in_repeated_calls(V, rows, noalloc):
    """Where the last workgroup of the row kernel sums the loss, its counter has to be zero again for the
    next call, whichever entry point and however many rows that has."""
    import paper_2410_10989_amd as flce
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    Z0 = (torch.randn(rows, V, device="cuda", generator=g)).to(torch.bfloat16)
    t = torch.randint(0, V, (rows,), device="cuda", generator=g)
    t[torch.rand(rows, device="cuda", generator=g) < 0.2] = -100
    lse = torch.logsumexp(Z0.double(), 1)
    for n in (rows, max(1, rows // 2), rows, rows):
        tn, ok = t[:n], t[:n] != -100
        want = float(((lse[:n] - Z0[:n].double().gather(1, tn.clamp(min=0)[:, None])[:, 0]) * ok).sum() / max(1, int(ok.sum())))
        loss = flce.flce_cross_entropy_inplace(Z0[:n].clone(), tn, -100, noalloc=noalloc)
        # a row's loss is a 32-bit number of size log V + |z| <= 20: rounded to 2^-20, some such steps in it
        assert abs(float(loss) - want) <= 1e-5, n
