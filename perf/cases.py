"""The work a user has this library do, through its public entry points: what is timed and
compared when a kernel or a host path changes.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from the seed alone
(hidden states ~ N(0, 1), head weights ~ N(0, 0.02^2), uniform or Zipf targets, a share of
ignored rows, logits ~ N(0, 1.3^2) for the stand-alone cross entropy), `run` is one pass,
`exact` the same result in plain torch in 64 bits.
"""
from __future__ import annotations

import torch

import paper_2410_10989_amd as flce

IGNORE = -100
EPS = 1e-6
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
MULTIHEAD_DECAY = 0.8   # loss weight of head j: 0.8^j
MULTIHEAD_SEQ = 512     # head j looks j tokens further on inside sequences of this length


def _case(name, entry, BT, H, V, dtype="bf16", targets="uniform", law="none", ignored=0.0, heads=1, skip="",
          ldz=0, noalloc=False):
    c = dict(entry=entry, BT=BT, H=H, V=V, dtype=dtype, targets=targets, law=law, ignored=ignored, heads=heads,
             skip=skip, ldz=ldz, noalloc=noalloc)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest training call: a toy head in fp32 (unit tests, debugging, tiny models);
        # launches and latency count
        _case("tiny_fp32", "fwd_bwd", 256, 512, 4096, "f32"),
        # a small model's head, natural-language-like (Zipf) targets, a few padded rows
        _case("small_zipf", "fwd_bwd", 1024, 512, 8192, targets="zipf", law="iid", ignored=0.05),
        # fine-tuning with a frozen head: a short, odd micro-batch against a full-size head,
        # only the hidden states' gradient is wanted
        _case("frozen_head_microbatch", "fwd_bwd", 200, 4096, 128256, law="iid", ignored=0.1, skip="dw"),
        # ordinary batches of the five benchmark heads' sizes
        _case("llama2_7b_head", "fwd_bwd", 4096, 4096, 32000, law="iid", ignored=0.10),
        _case("llama3_8b_head", "fwd_bwd", 8192, 4096, 128256, targets="zipf", law="iid", ignored=0.05),
        # the memory-pressure one: padded sequences, several chunks, dW summed over chunks
        _case("qwen2_7b_head", "fwd_bwd", 16384, 3584, 152064, law="pad", ignored=0.20),
        # the largest vocabulary, with the model's final RMSNorm in front of the head
        _case("gemma2_2b_rmsnorm_head", "rmsnorm", 8192, 2304, 256000, law="iid", ignored=0.30),
        # Medusa-style decoding heads on shared hidden states, trained jointly with the backbone
        _case("three_heads", "multihead", 2048, 4096, 32000, heads=3),
        # labels shifted by one (an odd row count), a hidden size that is no multiple of 64, a
        # GPT-2 vocabulary
        _case("ragged_bf16", "fwd_bwd", 2047, 1000, 50257, law="iid", ignored=0.1),
        # full-precision training of a GPT-2-medium-sized head
        _case("gpt2_fp32", "fwd_bwd", 2048, 1024, 50257, "f32", law="iid", ignored=0.1),
        # stand-alone cross entropy on logits another library made: a padded, aligned vocabulary ...
        _case("ce_bf16_122880", "ce", 4096, 1, 122880, law="iid", ignored=0.1, ldz=122880),
        # ... and the plain GPT-2 vocabulary, whose rows start at odd addresses, in a loop that
        # may not allocate
        _case("ce_bf16_50257", "ce", 4096, 1, 50257, law="iid", ignored=0.1, ldz=50257, noalloc=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """A case of the same ranges: 16 .. 16384 rows, hidden sizes 64 .. 4096 (multiples of 8, most
    of them of 64), vocabularies 257 .. 262144 of any residue, both storage types, every entry."""
    entry = rng.choice(["fwd_bwd"] * 4 + ["rmsnorm", "multihead", "ce", "ce"])
    dtype = "f32" if rng.random() < 0.3 else "bf16"
    law = rng.choice(["none", "iid", "iid", "pad"])
    ignored = 0.0 if law == "none" else 0.20 if law == "pad" else round(rng.uniform(0.02, 0.4), 3)
    BT = _log_uniform(rng, 16, 16384)
    if entry == "ce":
        V = _log_uniform(rng, 1000, 163840)
        if rng.random() < 0.5:
            V = (V + 63) // 64 * 64
        ldz = V if rng.random() < 0.5 else (V + 63) // 64 * 64
        BT = max(16, min(BT, (4096 * 122880) // V // (2 if dtype == "f32" else 1)))
        return _case("", "ce", BT, 1, V, dtype, law=law, ignored=ignored, ldz=ldz, noalloc=rng.random() < 0.3)
    step = 64 if rng.random() < 0.7 else 8
    H = max(64, _log_uniform(rng, 64, 4096) // step * step)
    V = _log_uniform(rng, 257, 262144)
    if rng.random() < 0.5:
        V = (V + 63) // 64 * 64
    heads = rng.choice([2, 3, 4]) if entry == "multihead" else 1
    # no dearer than the largest listed one: 4e13 operations in bf16; fp32 matrix instructions
    # run at a sixteenth of that rate
    most = (2.0e12 if dtype == "f32" else 3.0e13) / (6.0 * H * V * heads)
    BT = max(16, min(BT, int(most)))
    skip = rng.choice(["", "", "", "dx", "dw"]) if entry != "rmsnorm" else ""
    return _case("", entry, BT, H, V, dtype, rng.choice(["uniform", "zipf"]), law, ignored, heads, skip)


def _normal(g, shape, std, dtype):
    """N(0, std^2) rounded to `dtype`, in pieces (bounded temporaries)."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    piece = 1 << 26
    for s in range(0, flat.numel(), piece):
        n = min(piece, flat.numel() - s)
        flat[s:s + n] = torch.randn(n, generator=g, device="cuda") * std
    return out


def _make_targets(case, g):
    BT, V = case["BT"], case["V"]
    if case["targets"] == "zipf":   # Zipf(1.1) over ranks 1 .. V, class = rank - 1
        cdf = torch.cumsum(torch.arange(1, V + 1, dtype=torch.float64, device="cuda") ** -1.1, 0)
        u = torch.rand(BT, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
        t = torch.searchsorted(cdf, u).clamp_(max=V - 1)
    else:
        t = torch.randint(0, V, (BT,), generator=g, device="cuda")
    if case["law"] == "iid":
        t[torch.rand(BT, generator=g, device="cuda") < case["ignored"]] = IGNORE
    elif case["law"] == "pad":   # sequences of 2048 tokens that end in a run of padding
        pos = torch.arange(BT, device="cuda")
        run = (torch.rand((BT + 2047) // 2048, generator=g, device="cuda") * (2 * case["ignored"] * 2048)).long()
        t[pos % 2048 >= 2048 - run[pos // 2048]] = IGNORE
    return t


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(241010989 + 7919 * int(seed))
    BT, H, V, dt = case["BT"], case["H"], case["V"], DTYPES[case["dtype"]]
    s = {"t": _make_targets(case, g)}
    if case["entry"] == "ce":
        buf = _normal(g, (BT, case["ldz"]), 1.3, dt)
        s["Z"] = buf[:, :V]
        return s
    s["W"] = _normal(g, (V, H), 0.02, dt)
    s["X"] = _normal(g, (BT, H), 1.0, dt)
    if case["entry"] == "rmsnorm":   # raw hidden states: rows of different length; a learned scale
        s["X"] = (s["X"].float() * torch.exp(0.5 * torch.randn(BT, 1, generator=g, device="cuda"))).to(dt)
        s["gamma"] = (1.0 + 0.1 * torch.randn(H, generator=g, device="cuda")).to(dt)
    if case["entry"] == "multihead":
        n = case["heads"]
        s["Ws"] = [s["W"]] + [_normal(g, (V, H), 0.02, dt) for _ in range(1, n)]
        pos = torch.arange(BT, device="cuda")
        s["ts"] = []
        for j in range(n):
            tj = torch.roll(s["t"], -j)
            s["ts"].append(torch.where((pos % MULTIHEAD_SEQ + j < MULTIHEAD_SEQ) & (pos + j < BT), tj,
                                       torch.full_like(tj, IGNORE)))
        s["weights"] = [MULTIHEAD_DECAY ** j for j in range(n)]
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["flags"] = {"": 0, "dx": flce.SKIP_DX, "dw": flce.SKIP_DW}[case["skip"]]
    if case["entry"] == "ce":   # the loop that may not allocate brings its loss along
        s["loss"] = torch.empty((), dtype=torch.float32, device="cuda")
    return s


def run(s):
    """One pass.  The cross entropy turns its logits into their gradient in place: a further
    pass on the same state takes that gradient as logits, which costs the same."""
    c = s["case"]
    if c["entry"] == "ce":
        fn = flce.flce_cross_entropy_inplace_noalloc if c["noalloc"] else flce.flce_cross_entropy_inplace
        return [fn(s["Z"], s["t"], IGNORE, loss=s["loss"]), s["Z"]]
    if c["entry"] == "rmsnorm":
        return list(flce.flce_rmsnorm_fwd_bwd(s["X"], s["gamma"], EPS, s["W"], s["t"], IGNORE))
    if c["entry"] == "multihead":
        loss, head_losses, dX, dWs = flce.flce_multihead_fwd_bwd(s["X"], s["Ws"], s["ts"], s["weights"], IGNORE,
                                                                 flags=s["flags"])
        return [loss, head_losses, dX, dWs]
    return list(flce.flce_fwd_bwd(s["X"], s["W"], s["t"], IGNORE, flags=s["flags"]))


def work(case):
    """Rows with an ignored target need no arithmetic and, alone in the cross entropy, no read."""
    BT, H, V, n = case["BT"], case["H"], case["V"], case["heads"]
    es = 4 if case["dtype"] == "f32" else 2
    live = BT * (1.0 - case["ignored"])
    if case["entry"] == "ce":
        return {"bytes": (live + BT) * V * es + 8 * BT, "flops": 0}
    products = 2 if case["skip"] else 3
    want_dx, want_dw = case["skip"] != "dx", case["skip"] != "dw"
    return {"bytes": es * (BT * H * (1 + want_dx) + n * V * H * (1 + want_dw)) + 8 * n * BT,
            "flops": 2.0 * products * n * live * H * V}


def tolerance(case):
    """bf16: logits, their gradient and the results are each rounded to 8 bits on the way.
    fp32: sums of up to 262144 terms in 32 bits."""
    return {"rel": 2e-5 if case["dtype"] == "f32" else 1e-2}


def _xent64(z, t, n):
    """Loss sum and (softmax - onehot) / n of rows of logits in 64 bits; ignored rows give zeros."""
    ok = t != IGNORE
    at = t.clamp(min=0)[:, None]
    lse = torch.logsumexp(z, 1, keepdim=True)
    loss = ((lse - z.gather(1, at))[:, 0] * ok).sum()
    g = torch.exp(z - lse)
    g.scatter_add_(1, at, torch.full_like(lse, -1.0))
    g *= (ok.double() / max(1, n))[:, None]
    return loss, g


def _head64(X, W, t, want_dx, want_dw):
    n = int((t != IGNORE).sum())
    W = W.double()
    loss = torch.zeros((), dtype=torch.float64, device="cuda")
    dX = torch.zeros_like(X) if want_dx else None
    dW = torch.zeros_like(W) if want_dw else None
    step = max(64, (1 << 28) // W.shape[0])   # 2 GiB of logits at a time
    for r in range(0, X.shape[0], step):
        x = X[r:r + step]
        part, g = _xent64(x @ W.T, t[r:r + step], n)
        loss += part
        if want_dx:
            dX[r:r + step] = g @ W
        if want_dw:
            dW += g.T @ x
    return loss / max(1, n), dX, dW


def exact(case, seed):
    s = _inputs(case, seed)
    if case["entry"] == "ce":
        Z, t, V = s["Z"], s["t"], case["V"]
        n = int((t != IGNORE).sum())
        loss = torch.zeros((), dtype=torch.float64, device="cuda")
        out = torch.empty(Z.shape, dtype=torch.float64, device="cuda")
        step = max(1, (1 << 28) // V)
        for r in range(0, Z.shape[0], step):
            part, out[r:r + step] = _xent64(Z[r:r + step].double(), t[r:r + step], n)
            loss += part
        return [loss / max(1, n), out]
    want_dx, want_dw = case["skip"] != "dx", case["skip"] != "dw"
    X = s["X"].double()
    if case["entry"] == "rmsnorm":
        rms = torch.sqrt((X * X).mean(1, keepdim=True) + EPS)
        xhat, gamma = X / rms, s["gamma"].double()
        loss, dY, dW = _head64(xhat * gamma, s["W"], s["t"], True, True)
        a = dY * gamma
        dh = (a - (xhat * a).mean(1, keepdim=True) * xhat) / rms
        return [loss, dh, (dY * xhat).sum(0), dW]
    if case["entry"] == "multihead":
        total = torch.zeros((), dtype=torch.float64, device="cuda")
        means, dX, dWs = [], torch.zeros_like(X), []
        for W, t, w in zip(s["Ws"], s["ts"], s["weights"]):
            loss, dx, dw = _head64(X, W, t, want_dx, want_dw)
            total += w * loss
            means.append(loss)
            if want_dx:
                dX += w * dx
            if want_dw:
                dWs.append(w * dw)
        return [total, torch.stack(means), dX if want_dx else None, dWs if want_dw else None]
    return list(_head64(X, s["W"], s["t"], want_dx, want_dw))
