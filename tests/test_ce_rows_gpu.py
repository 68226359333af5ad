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


def _small_batch(rows, V, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    Z = torch.randn(rows, V, device="cuda", generator=g).to(torch.bfloat16)
    t = torch.randint(0, V, (rows,), device="cuda", generator=g)
    t[torch.rand(rows, device="cuda", generator=g) < 0.2] = -100
    ok = t != -100
    lse = torch.logsumexp(Z.double(), 1)
    return Z, t, float(((lse - Z.double().gather(1, t.clamp(min=0)[:, None])[:, 0]) * ok).sum() / max(1, int(ok.sum())))


def _on_two_streams(calls):
    """calls[j]: what stream j does; both start together, once some milliseconds of other work have ended."""
    gate, streams = torch.cuda.Stream(), [torch.cuda.Stream() for _ in calls]
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(gate):
        for _ in range(20):
            busy @ busy
        opened = gate.record_event()
    for s, todo in zip(streams, calls):
        s.wait_event(opened)
        with torch.cuda.stream(s):
            for call in todo:
                call()
    torch.cuda.synchronize()


def test_small_batches_that_overlap_on_lent_buffers():
    # calls on different lent buffers share nothing: 100 calls on each of two streams at the same time
    import paper_2410_10989_amd as flce
    n, sizes = 100, ((300, 30000), (190, 30000))
    buffers = [torch.empty(1 << 16, dtype=torch.uint8, device="cuda") for _ in sizes]
    data = [[_small_batch(*size, 31 * j + k) for k in range(3)] for j, size in enumerate(sizes)]
    Zs = [[data[j][k % 3][0].clone() for k in range(n)] for j in range(2)]
    losses = [torch.full((n,), float("nan"), device="cuda") for _ in sizes]

    def call(j, k):
        flce.flce_set_workspace(buffers[j])
        flce.flce_cross_entropy_inplace(Zs[j][k], data[j][k % 3][1], -100, loss=losses[j][k])

    try:
        _on_two_streams([[lambda j=j, k=k: call(j, k) for k in range(n)] for j in range(2)])
    finally:
        flce.flce_set_workspace(None)
    for j in range(2):
        want = torch.tensor([data[j][k % 3][2] for k in range(n)])
        assert float((losses[j].cpu().double() - want.double()).abs().max()) <= 1e-5, j   # as above


def test_small_batches_after_calls_that_overlapped():
    # overlapping calls of the allocation-free entry point are forbidden and their results open; the calls after
    # them are right again
    import paper_2410_10989_amd as flce
    n = 100
    data = [_small_batch(rows, 30000, rows) for rows in (300, 190)]
    Zs = [[d[0].clone() for _ in range(n)] for d in data]
    out = torch.empty(2 * n, device="cuda")
    _on_two_streams([[lambda j=j, k=k: flce.flce_cross_entropy_inplace_noalloc(Zs[j][k], data[j][1], -100, loss=out[j * n + k])
                      for k in range(n)] for j in range(2)])
    for rows in (300, 17, 512, 33, 1, 300):
        Z, t, want = _small_batch(rows, 3000, rows)
        loss = torch.full((), float("nan"), device="cuda")
        flce.flce_cross_entropy_inplace_noalloc(Z, t, -100, loss=loss)
        assert abs(float(loss) - want) <= 1e-5, rows



@pytest.mark.parametrize("noalloc", [False, True])
def test_captured_small_batches_beside_eager_ones(noalloc):
    # a replay repeats its launches' arguments: captured calls sum the loss in a launch of its own
    import paper_2410_10989_amd as flce
    Z0, t, want = _small_batch(100, 3000, 5)
    Z, loss = Z0.clone(), torch.full((), float("nan"), device="cuda")
    flce.flce_cross_entropy_inplace(Z0.clone(), t, -100, noalloc=noalloc)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        flce.flce_cross_entropy_inplace(Z, t, -100, loss=loss, noalloc=noalloc)
    for k in range(4):
        Z.copy_(Z0)
        loss.fill_(float("nan"))
        graph.replay()
        eager = Z0.clone()
        loss_eager = flce.flce_cross_entropy_inplace(eager, t, -100, noalloc=noalloc)
        torch.cuda.synchronize()
        assert abs(float(loss) - want) <= 1e-5 and float(loss) == float(loss_eager), k
        assert torch.equal(Z, eager), k
