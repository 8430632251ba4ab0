"""The work that a program built on this library has it do, as cases that can be timed and compared.

Three kinds of pass, each through the public entry points:

* "round": one verify round of speculative decoding over a stack of layers.  Per layer the fused conv roll, replay, draft
  scan and snapshots (ssm_conv_verify_multistep, or ssm_block_multistep where the step-size transform, the gate or ragged
  draft counts are asked for; "norm": followed by ssmv_gated_rmsnorm), then FirstConflict on the round's tokens and one
  commit over all layers.  "graph": the round is captured once and replayed, as a decoder does that runs the same round
  again and again; without it every call goes through the binding.
* "draft": the draft side of such a round: k single-token calls per layer that recompute from the cached state.
* "prefill": a prompt through one layer, and the state taken out row-major as it is handed to another engine.  "resume":
  the prompt continues a sequence (chunked feeding); without it the cache is reset first, as for a new request.

The caches of "round" and "draft" are two rounds old when a pass starts, so that the pending counts have the mix of a
running decoder (on a fresh cache nothing is pending).  Distributions are those of `workload`: x ~ N(0,1), B, C ~
N(0,1)/sqrt(dstate), dt = softplus(N(0,1) - 4), A = -exp(U(0, ln 16)) per head or -(n+1) + U(-1/4, 1/4) per channel.
"""
from __future__ import annotations

import math

import torch

import paper_2408_15237_amd as ssmv

IO = {"bf16": torch.bfloat16, "f32": torch.float32}
PRIMED = 2              # rounds a decoder has behind it when a pass starts
GEOMETRIC_REJECT = 0.3  # chance that a draft token is rejected ("geometric" acceptance)
EPS = 1e-5

_ROUND = dict(kind="round", io="bf16", mode="scalar", batch=1, heads=32, headdim=128, dstate=64, groups=1, k=4, layers=24,
              accept="uniform", snapshot="both", act="none", softplus=False, gate=False, norm=False, ragged=False, graph=True)
_PREFILL = dict(kind="prefill", io="bf16", batch=1, heads=32, headdim=128, dstate=64, groups=1, length=2048, act="none",
                softplus=False, gate=False, norm=False, ragged=False, resume=False)


def listed():
    return [
        # a first integration: the tiny fp32 layer, one call after another through the binding
        dict(_ROUND, name="round_tiny_f32", io="f32", heads=4, headdim=16, dstate=16, layers=1, graph=False),
        # one user, an 8B-shaped hybrid: latency of a round over all its SSM layers
        dict(_ROUND, name="round_8b_b1"),
        # one user, a Mamba-1 style model (a decay per channel and state index), long drafts
        dict(_ROUND, name="round_mamba1_b1", mode="diag", heads=8192, headdim=1, dstate=16, k=8, accept="geometric"),
        # a serving batch of the 8B shape
        dict(_ROUND, name="round_8b_b32", batch=32, layers=4),
        # a serving batch with long drafts and the whole block's recurrence: softplus, conv SiLU, gate, norm
        dict(_ROUND, name="round_block_b16", batch=16, k=8, layers=8, act="silu", softplus=True, gate=True, norm=True),
        # a serving batch of the Mamba-1 style model, every sequence with a draft count of its own
        dict(_ROUND, name="round_mamba1_b24", mode="diag", batch=24, heads=5120, headdim=1, dstate=16, k=6, layers=4, act="silu",
             softplus=True, ragged=True, accept="geometric"),
        # fp32 tensors, grouped B and C, the single-snapshot variant
        dict(_ROUND, name="round_f32_b6", io="f32", batch=6, heads=80, headdim=64, dstate=128, groups=8, layers=4, snapshot="hj_only"),
        # the draft model's side of a serving round on caches with a deferred advance
        dict(_ROUND, name="draft_b32", kind="draft", batch=32, layers=4, snapshot="defer"),
        # prompts of a full batch
        dict(_PREFILL, name="prefill_b32", batch=32),
        # one prompt of an ordinary length, continuing a conversation
        dict(_PREFILL, name="prefill_b1", length=1500, resume=True),
        # a few prompts of different lengths through a whole block: softplus, conv SiLU, gate, norm, grouped B and C
        dict(_PREFILL, name="prefill_block_b5", batch=5, heads=80, headdim=64, dstate=128, groups=8, length=700, act="silu", softplus=True,
             gate=True, norm=True, ragged=True),
        # fp32 tensors, a small batch
        dict(_PREFILL, name="prefill_f32_b4", io="f32", batch=4, length=1021, resume=True),
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _groups(rng, heads):
    return rng.choice([g for g in (1, 1, 2, 4, 8) if heads % g == 0])


def draw(rng):
    kind = rng.choice(["round", "round", "diag", "draft", "prefill", "prefill", "prefill_f32"])
    if kind in ("round", "draft"):
        io = "bf16" if kind == "draft" else rng.choice(["bf16", "bf16", "f32"])
        heads = _log_int(rng, 4, 80)
        headdim = rng.choice([64, 128]) if kind == "draft" else rng.choice([16, 32, 64, 64, 128, 128])
        dstate = rng.choice([32, 64, 128]) if kind == "draft" else rng.choice([16, 32, 64, 64, 128, 256])
        k = rng.randint(2, 8)
        elems = heads * headdim * dstate
        # one serving batch of the listed shape holds 2^23 state values per layer
        batch = _log_int(rng, 1, max(1, min(32, (1 << 23) // elems)))
        return dict(_ROUND, kind=kind, io=io, batch=batch, heads=heads, headdim=headdim, dstate=dstate, groups=_groups(rng, heads), k=k,
                    layers=rng.randint(2, 4 if batch > 4 else 16), snapshot=rng.choice(["both", "both", "hj_only", "defer"]),
                    act=rng.choice(["none", "silu"]), softplus=rng.random() < 0.5, gate=kind == "round" and rng.random() < 0.5,
                    ragged=kind == "round" and rng.random() < 0.3)
    if kind == "diag":
        heads = 16 * _log_int(rng, 32, 512)
        dstate = rng.choice([16, 16, 16, 32])
        return dict(_ROUND, mode="diag", io=rng.choice(["bf16", "bf16", "f32"]), batch=_log_int(rng, 1, max(1, min(32, (1 << 21) // (heads * dstate // 2)))),
                    heads=heads, headdim=1, dstate=dstate, k=rng.randint(2, 8), layers=rng.randint(2, 8), accept="geometric",
                    act=rng.choice(["none", "silu"]), softplus=rng.random() < 0.5, ragged=rng.random() < 0.3)
    heads = _log_int(rng, 4, 80)
    headdim, dstate = rng.choice([32, 64, 64, 128, 128]), rng.choice([32, 64, 64, 128])
    # tokens of all sequences together: never more work than the listed full batch (fp32 products: an eighth of it)
    most = (65536 if kind == "prefill" else 8192) * (32 * 128 * 64) // (heads * headdim * dstate)
    length = _log_int(rng, 1, min(4096, most))
    batch = _log_int(rng, 1, max(1, min(32, most // length)))
    return dict(_PREFILL, io="bf16" if kind == "prefill" else "f32", batch=batch, heads=heads, headdim=headdim, dstate=dstate,
                groups=_groups(rng, heads), length=length, act=rng.choice(["none", "silu"]), softplus=rng.random() < 0.5,
                gate=rng.random() < 0.5, ragged=batch > 1 and rng.random() < 0.5, resume=rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------------------------------------


def _generator(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what) % (1 << 62))
    return g


def _layer(c, seed, layer):
    """Parameters of one layer and what its cache starts from."""
    g, io = _generator(seed, 7919 * (layer + 1)), IO[c["io"]]
    H, P, N, b = c["heads"], c["headdim"], c["dstate"], c["batch"]
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    if c.get("mode", "scalar") == "diag":
        A = -(torch.arange(1, N + 1, device="cuda", dtype=torch.float32) + (rand(H, N) - 0.5) * 0.5)
    else:
        A = -torch.exp(rand(H) * math.log(16.0))
    return dict(A=A.contiguous(), D=randn(H), w=(randn(H * P, 4) / 2).to(io), bias=(randn(H * P) * 0.1).to(io),
                h0=(randn(b, H, P, N) * 0.1), conv=randn(b, 3, H * P).to(io), dt_bias=rand(H) - 0.5, norm=1 + 0.1 * randn(H * P))


def _tokens(c, seed, layer, n, what):
    """The n tokens of every sequence that one call takes."""
    g, io = _generator(seed, 104729 * (layer + 1) + what), IO[c["io"]]
    b, H, Cx, G, N = c["batch"], c["heads"], c["heads"] * c["headdim"], c["groups"], c["dstate"]
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    dt = randn(b, n, H) - 4.0
    return dict(x=randn(b, n, Cx).to(io), dt=(dt if c["softplus"] else torch.nn.functional.softplus(dt)).to(io), B=(randn(b, n, G, N) / N ** 0.5).to(io),
                C=(randn(b, n, G, N) / N ** 0.5).to(io), z=randn(b, n, Cx).to(io) if c["gate"] or c["norm"] else None)


def _drafts(c, seed, rnd):
    """Draft tokens, the target's tokens, and how many of each sequence's drafts are looked at."""
    g = torch.Generator().manual_seed(int(seed) * 31 + rnd)
    b, k = c["batch"], c["k"]
    if c["accept"] == "uniform":
        acc = torch.randint(0, k + 1, (b,), generator=g)
    else:
        acc = (torch.log(1 - torch.rand(b, generator=g)) / math.log(1 - GEOMETRIC_REJECT)).long().clamp(0, k)
    counts = torch.randint(1, k + 1, (b,), generator=g) if c["ragged"] else torch.full((b,), k)
    acc = torch.minimum(acc, counts)
    draft = torch.randint(0, 32000, (b, k), generator=g)
    target = draft.clone()
    wrong = acc < k
    target[wrong, acc[wrong]] += 1
    return draft.int().cuda(), target.int().cuda(), counts.int().cuda()


def _dims(c):
    k = c.get("k", 4)
    return ssmv.make_dims(c["batch"], c["heads"], c["headdim"], c["dstate"], ngroups=c["groups"], kmax=k, io=c["io"],
                          a_mode=c.get("mode", "scalar"), conv_act=c["act"], snapshot_mode=c.get("snapshot", "both"))


def _cache(dims, p):
    cache = ssmv.LayerCache.allocate(dims)
    ssmv.ssmv_cache_reset(dims, cache.c, p["h0"], p["conv"])
    return cache


# ---- rounds --------------------------------------------------------------------------------------------------------------


def _verify(s, layer, tok, counts):
    """One layer's verify call."""
    c, p, dims, cache, y = s["case"], s["layers"][layer], s["dims"], s["caches"][layer].c, s["y"][layer]
    if c["softplus"] or c["gate"] or c["ragged"]:
        ssmv.ssm_block_multistep(dims, cache, x_raw=tok["x"], conv_wgt=p["w"], conv_bias=p["bias"], dt=tok["dt"],
                                 dt_bias=p["dt_bias"] if c["softplus"] else None, dt_softplus=c["softplus"], Bm=tok["B"], Cm=tok["C"],
                                 z=tok["z"] if c["gate"] else None, A=p["A"], D=p["D"], k=c["k"], k_seq=counts if c["ragged"] else None, y_out=y)
    else:
        ssmv.ssm_conv_verify_multistep(dims, cache, tok["x"], p["w"], p["bias"], tok["dt"], tok["B"], tok["C"], p["A"], p["D"], c["k"], y)
    if c["norm"]:
        rows, channels = c["batch"] * c["k"], c["heads"] * c["headdim"]
        ssmv.ssmv_gated_rmsnorm(y, None if c["gate"] else tok["z"], p["norm"], rows, channels, channels // c["groups"], EPS, c["io"], s["normed"][layer])


def _draft(s, layer, tok):
    """One layer's k single-token calls: each recomputes from the cached state, the last one stores the snapshots."""
    c, p, dims, cache = s["case"], s["layers"][layer], s["dims"], s["caches"][layer].c
    for t in range(c["k"]):
        ssmv.ssm_block_multistep(dims, cache, x_raw=tok["x"][t], conv_wgt=p["w"], conv_bias=p["bias"], dt=tok["dt"][t],
                                 dt_bias=p["dt_bias"] if c["softplus"] else None, dt_softplus=c["softplus"], Bm=tok["B"][t], Cm=tok["C"][t],
                                 A=p["A"], D=p["D"], k=1, tok0=t, y_out=s["y"][layer][t], replay_round=True, last_call=t == c["k"] - 1)


def _round(s, tokens, drafts):
    c = s["case"]
    draft, target, counts = drafts
    for layer in range(c["layers"]):
        if c["kind"] == "draft":
            _draft(s, layer, tokens[layer])
        else:
            _verify(s, layer, tokens[layer], counts)
    ssmv.ssmv_first_conflict(draft, target, c["batch"], c["k"], s["accepted"])
    ssmv.ssm_commit_rollback_multi(s["dims"], s["cache_structs"], s["accepted"])


def _round_tokens(c, seed, rnd):
    """Per layer the tokens of round `rnd`; for the draft side one contiguous set per call."""
    out = []
    for layer in range(c["layers"]):
        tok = _tokens(c, seed, layer, c["k"], rnd)
        if c["kind"] == "draft":
            tok = {n: None if v is None else [v[:, t:t + 1].contiguous() for t in range(c["k"])] for n, v in tok.items()}
        out.append(tok)
    return out


def _prepare_round(c, seed):
    io, b, k, Cx, n = IO[c["io"]], c["batch"], c["k"], c["heads"] * c["headdim"], c["layers"]
    dims = _dims(c)
    layers = [_layer(c, seed, i) for i in range(n)]
    caches = [_cache(dims, p) for p in layers]
    shape = (n, k, b, 1, Cx) if c["kind"] == "draft" else (n, b, k, Cx)
    s = dict(case=c, dims=dims, layers=layers, caches=caches, cache_structs=(ssmv.ssmv_cache * n)(*[x.c for x in caches]),
             y=torch.zeros(shape, dtype=io, device="cuda"), normed=torch.zeros(shape, dtype=io, device="cuda") if c["norm"] else None,
             accepted=torch.zeros(b, dtype=torch.int32, device="cuda"))
    for p in layers:
        del p["h0"], p["conv"]
    for rnd in range(PRIMED):
        _round(s, _round_tokens(c, seed, rnd), _drafts(c, seed, rnd))
    s["tokens"], s["drafts"] = _round_tokens(c, seed, PRIMED), _drafts(c, seed, PRIMED)
    if c["graph"]:
        torch.cuda.synchronize()
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            graph.capture_begin()
            _round(s, s["tokens"], s["drafts"])
            graph.capture_end()
        torch.cuda.synchronize()
        s["graph"] = graph
    return s


def _run_round(s):
    if "graph" in s:
        s["graph"].replay()
    else:
        _round(s, s["tokens"], s["drafts"])
    return dict(y=s["normed"] if s["case"]["norm"] else s["y"], accepted=s["accepted"], pend=s["caches"][0].buffers["pend"],
                pos=s["caches"][0].buffers["pos"], state=[x.state_view() for x in s["caches"]])


# ---- prefill -------------------------------------------------------------------------------------------------------------


def _lengths(c, seed):
    """Prompt lengths: the longest is c["length"]; ragged prompts from one token up."""
    g = torch.Generator().manual_seed(int(seed) * 17 + 3)
    n = torch.randint(1, c["length"] + 1, (c["batch"],), generator=g) if c["ragged"] else torch.full((c["batch"],), c["length"])
    n[0] = c["length"]
    return n


def _prepare_prefill(c, seed):
    dims, p, tok = _dims(c), _layer(c, seed, 0), _tokens(c, seed, 0, c["length"], 0)
    y = torch.zeros_like(tok["x"])
    return dict(case=c, dims=dims, layer=p, tok=tok, cache=_cache(dims, p), y=y, normed=torch.zeros_like(y) if c["norm"] else None,
                lens=_lengths(c, seed).int().cuda() if c["ragged"] else None, h=torch.empty_like(p["h0"]))


def _run_prefill(s):
    c, p, tok, dims, cache = s["case"], s["layer"], s["tok"], s["dims"], s["cache"].c
    if not c["resume"]:
        ssmv.ssmv_cache_reset(dims, cache)
    bias = p["dt_bias"] if c["softplus"] else None
    if c["softplus"] or c["gate"] or c["ragged"]:
        ssmv.ssm_prefill_block(dims, cache, x_raw=tok["x"], conv_wgt=p["w"], conv_bias=p["bias"], dt=tok["dt"], dt_bias=bias, dt_softplus=c["softplus"],
                               Bm=tok["B"], Cm=tok["C"], z=tok["z"] if c["gate"] else None, A=p["A"], D=p["D"], L=c["length"], y_out=s["y"],
                               seq_len=s["lens"])
    else:
        ssmv.ssm_prefill_chunked(dims, cache, tok["x"], p["w"], p["bias"], tok["dt"], tok["B"], tok["C"], p["A"], p["D"], c["length"], s["y"])
    y = s["y"]
    if c["norm"]:
        y, channels = s["normed"], c["heads"] * c["headdim"]
        ssmv.ssmv_gated_rmsnorm(s["y"], None if c["gate"] else tok["z"], p["norm"], c["batch"] * c["length"], channels, channels // c["groups"], EPS, c["io"], y)
    ssmv.ssmv_materialize_block(dims, cache, p["A"], bias, c["softplus"], s["h"])
    return dict(y=y, state=s["h"])


def prepare(case, seed):
    return _prepare_prefill(case, seed) if case["kind"] == "prefill" else _prepare_round(case, seed)


def run(state):
    return _run_prefill(state) if state["case"]["kind"] == "prefill" else _run_round(state)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------


def work(case):
    c = case
    e = 2 if c["io"] == "bf16" else 4
    b, H, P, N, G = c["batch"], c["heads"], c["headdim"], c["dstate"], c["groups"]
    Cx, elems = H * P, c["batch"] * H * P * N
    # per state value and token: the decay, the outer product into it, the contraction out of it
    per_token = 5 * H * P * N
    gated = 1 if c["gate"] or c["norm"] else 0
    if c["kind"] == "prefill":
        n = c["length"] * ((b + 1) / 2 if c["ragged"] else b)                   # mean length of ragged prompts: half the longest
        by = n * ((2 + gated) * Cx + H + 2 * G * N) * e + Cx * 5 * e + elems * 4 * (2 if c["resume"] else 1)
        return {"bytes": by, "flops": n * (per_token + 8 * Cx)}
    k = c["k"]
    if c["ragged"]:
        k = (k + 1) / 2
    mean_pend = k / 2 if c["accept"] == "uniform" else min(k, 2.3)
    if c["snapshot"] == "both":
        # h_k always; h_j where tokens are pending
        stored = 1 + ((c["k"] - 1) / (c["k"] + 1) if c["accept"] == "uniform" else 0.65)
    elif c["snapshot"] == "hj_only":
        stored = c["k"] / (c["k"] + 1)
    else:
        # a stored state takes in the tokens that have collected behind the live one
        stored = min(1.0, mean_pend / max(1.0, 16 - 2 * c["k"] + mean_pend))
    tokens = k * ((2 + gated) * Cx + H + 2 * G * N) + k * (2 * Cx + H + G * N) + mean_pend * (Cx + H + G * N) + 3 * Cx
    per_layer = elems * 4 * (1 + stored) + b * tokens * e + Cx * 5 * e
    return {"bytes": c["layers"] * per_layer, "flops": c["layers"] * b * (k + mean_pend) * (per_token + 8 * Cx)}


def tolerance(case):
    if case["io"] == "bf16":
        # outputs are rounded to bf16 (2^-9 at most, a third of it on average), prefill multiplies bf16 heads
        return {"rel": 1e-2, "max": 0.2}
    return {"rel": 4e-6, "max": 2e-4}


# ---- the same in 64 bits, token by token --------------------------------------------------------------------------------


class _Exact:
    """The recurrence of one layer in 64 bits, from the definition: the state after the accepted tokens and the last three
    raw inputs; one token at a time."""

    def __init__(self, c, p, zero):
        d = lambda t: t.double()
        self.c, self.diag, self.io = c, c.get("mode", "scalar") == "diag", IO[c["io"]]
        self.A, self.D, self.w, self.bias, self.dt_bias, self.norm = (d(p[n]) for n in ("A", "D", "w", "bias", "dt_bias", "norm"))
        self.h = torch.zeros_like(p["h0"], dtype=torch.float64) if zero else d(p["h0"])
        self.hist = torch.zeros_like(p["conv"], dtype=torch.float64) if zero else d(p["conv"])

    def tokens(self, tok, n, keep):
        """Outputs of the first n tokens; sequence i keeps the state after its first keep[i]."""
        c = self.c
        b, H, P, N, G = c["batch"], c["heads"], c["headdim"], c["dstate"], c["groups"]
        raw = torch.cat([self.hist, tok["x"][:, :n].double()], dim=1)
        y = torch.zeros(b, n, H * P, dtype=torch.float64, device="cuda")
        h, kept = self.h, self.h.clone()
        hist = self.hist.clone()
        reach = [int(v) for v in keep]
        for t in range(n):
            xc = (raw[:, t:t + 4].transpose(1, 2) * self.w).sum(-1) + self.bias
            if c["act"] == "silu":
                xc = xc * torch.sigmoid(xc)
            xc = xc.to(self.io).double()                     # the conv output is a stored activation: its rounding is part of the definition
            dt = tok["dt"][:, t].double()
            if c["softplus"]:
                dt = torch.nn.functional.softplus(dt + self.dt_bias, threshold=50)
            Bt, Ct = (tok[m][:, t].double().repeat_interleave(H // G, dim=1) if not self.diag else tok[m][:, t].double() for m in ("B", "C"))
            x = xc.view(b, H, P)
            decay = torch.exp(dt[:, :, None] * self.A)[:, :, None, :] if self.diag else torch.exp(dt * self.A)[:, :, None, None]
            h = h * decay + (dt[:, :, None] * x)[:, :, :, None] * Bt[:, :, None, :]
            out = (h * Ct[:, :, None, :]).sum(-1) + self.D[:, None] * x
            out = out.reshape(b, H * P)
            if c["gate"]:
                zt = tok["z"][:, t].double()
                out = out * zt * torch.sigmoid(zt)
            y[:, t] = out
            at = [i for i, r in enumerate(reach) if r == t + 1]
            if at:
                kept[at] = h[at]
                hist[at] = raw[at, t + 1:t + 4]
        self.h, self.hist = kept, hist
        return y

    def normed(self, y, tok, n):
        if not self.c["norm"]:
            return y
        g = y
        if not self.c["gate"]:
            z = tok["z"][:, :n].double()
            g = y * z * torch.sigmoid(z)
        shape = g.shape[:2] + (self.c["groups"], -1)
        g = g.reshape(shape)
        return (g * torch.rsqrt((g * g).mean(-1, keepdim=True) + EPS)).reshape(y.shape) * self.norm


def exact(case, seed):
    c = case
    if c["kind"] == "prefill":
        n, p = c["length"], _layer(c, seed, 0)
        if c["batch"] * c["heads"] * c["headdim"] * c["dstate"] * n > 3e10:
            return None                                      # over about 20 seconds
        tok, lens = _tokens(c, seed, 0, n, 0), _lengths(c, seed)
        m = _Exact(c, p, not c["resume"])
        y = m.tokens(tok, n, lens)
        y[torch.arange(n)[None, :] >= lens[:, None]] = 0.0    # behind a sequence's length nothing is written
        return dict(y=m.normed(y, tok, n), state=m.h)
    k, ys = c["k"], []
    for layer in range(c["layers"]):
        p = _layer(c, seed, layer)
        m = _Exact(c, p, False)
        for rnd in range(PRIMED + 1):
            draft, target, counts = (t.cpu() for t in _drafts(c, seed, rnd))
            acc = (draft == target).int().cumprod(1).sum(1)
            tok = _tokens(c, seed, layer, k, rnd)
            y = m.tokens(tok, k, acc)
            y[torch.arange(k)[None, :] >= counts[:, None]] = 0.0
        ys.append(m.normed(y, tok, k))
    y = torch.stack(ys)
    if c["kind"] == "draft":
        y = y.permute(0, 2, 1, 3).unsqueeze(3).contiguous()
    return dict(y=y, accepted=None, pend=None, pos=None, state=None)
