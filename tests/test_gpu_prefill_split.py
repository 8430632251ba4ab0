"""GPU parity of prompts that are cut into segments (csrc/prefill_split.h): few (sequence, head) pairs and a prompt long
enough, so that the launch would leave most of the chip idle.  Every tile shape; lengths at the edges of chunks and
segments; sequences of one call that are cut into many segments, two, one, or none at all."""
import ctypes
import dataclasses
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2408_15237_amd as ssmv
from workload import Workload, generate, round_to_io

from _harness import HipLayer, TOL, launches, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [(P, N) for P in (32, 64, 128) for N in (32, 64, 128)]


def _inputs(io, P, N, H, G, batch, L, act="none", seed=11):
    dec = Workload("split", "scalar", batch=batch, nheads=H, headdim=P, dstate=N, k=4, rounds=2, io=io, accept="uniform", ngroups=G,
                   conv_act=act, seed=seed)
    data = generate(dec)
    rng = np.random.default_rng(seed + 1)
    draw = lambda *s: round_to_io(np.asarray(rng.standard_normal(s), dtype=np.float32), io)
    tok = dict(x=draw(batch, L, H * P), dt=round_to_io(rng.standard_normal((batch, L, H)) - 4.0, io), z=draw(batch, L, H * P),
               B=round_to_io(rng.standard_normal((batch, L, G, N)) / np.sqrt(N), io), C=round_to_io(rng.standard_normal((batch, L, G, N)) / np.sqrt(N), io))
    bias = rng.uniform(-0.5, 0.5, size=H).astype(np.float32)
    return dec, data, data.layers[0], tok, bias, draw(batch, 3, H * P)


def _prefill(hip, tok, bias, io, L, y, z, lens=None):
    ssmv.ssm_prefill_block(hip.dims, hip.cache.c, x_raw=to_dev(tok["x"], io), conv_wgt=hip.conv_w, conv_bias=hip.conv_b, dt=to_dev(tok["dt"], io),
                           dt_bias=torch.from_numpy(bias).to("cuda"), dt_softplus=True, Bm=to_dev(tok["B"], io), Cm=to_dev(tok["C"], io), z=z,
                           A=hip.A, D=hip.D, L=L, y_out=y, seq_len=None if lens is None else torch.from_numpy(lens).to("cuda"))


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("P,N", SHAPES)
def test_segments_of_ragged_prompts_then_decoding(P, N, io):
    H, G, L = 4, 2, 1200
    lens = np.array([L, 0, 1, 33, L - 31, 32 * 20, 32 * 12 + 1], dtype=np.int32)
    batch = len(lens)
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, G, batch, L, act="silu" if P == 64 else "none")
    hip = HipLayer(dec, lp, conv_init=conv_init)
    y = torch.full((batch, L, H * P), 7.0, dtype=torch.bfloat16 if io == "bf16" else torch.float32, device="cuda")
    _prefill(hip, tok, bias, io, L, y, to_dev(tok["z"], io), lens)
    y_h, h_g, ints = to_host(y), to_host(_materialize(hip, bias)), hip.cache.ints()
    oras = []
    for b, n in enumerate(int(v) for v in lens):
        ora = oracle.EagerOracle("scalar", lp.A, lp.D, lp.conv_w, lp.conv_b, lp.h0[b:b + 1], io, dec.conv_act, G, dt_bias=bias, dt_softplus=True,
                                 conv_init=conv_init[b:b + 1])
        if n:
            y_ref, _, _ = ora.verify(tok["x"][b:b + 1, :n], tok["dt"][b:b + 1, :n], tok["B"][b:b + 1, :n], tok["C"][b:b + 1, :n], z=tok["z"][b:b + 1, :n])
            ora.commit([n])
            assert rel_err(y_h[b, :n], y_ref[0]) <= TOL[io], "sequence %d" % b
        assert np.all(y_h[b, n:] == 7.0), "sequence %d: outputs behind its length were written" % b
        assert rel_err(h_g[b:b + 1], ora.h) <= TOL[io], "sequence %d: state" % b
        oras.append(ora)
    assert ints["pos"].tolist() == lens.tolist() and ints["err_flag"] == 0 and ints["pend"].tolist() == [0] * batch
    assert ints["conv_head"].tolist() == [(2 + int(n)) & (dec.ring_len - 1) for n in lens]
    rd = data.rounds[0]                                       # the ring and the state continue the prompt
    y_g = torch.empty_like(to_dev(rd.x_raw, io))
    dt = round_to_io(np.random.default_rng(5).standard_normal((batch, dec.k, H)) - 4.0, io)
    ssmv.ssm_block_multistep(hip.dims, hip.cache.c, x_raw=to_dev(rd.x_raw, io), conv_wgt=hip.conv_w, conv_bias=hip.conv_b, dt=to_dev(dt, io),
                             dt_bias=torch.from_numpy(bias).to("cuda"), dt_softplus=True, Bm=to_dev(rd.B[0], io), Cm=to_dev(rd.C[0], io), A=hip.A,
                             D=hip.D, k=dec.k, y_out=y_g)
    for b in range(batch):
        y_r, _, _ = oras[b].verify(rd.x_raw[b:b + 1], dt[b:b + 1], rd.B[0][b:b + 1], rd.C[0][b:b + 1])
        assert rel_err(to_host(y_g)[b:b + 1], y_r) <= TOL[io], "decode, sequence %d" % b


def _materialize(hip, bias):
    wl = hip.wl
    h = torch.empty((wl.batch, wl.nheads, wl.headdim, wl.dstate), dtype=torch.float32, device="cuda")
    ssmv.ssmv_materialize_block(hip.dims, hip.cache.c, hip.A, torch.from_numpy(bias).to("cuda"), True, h)
    return h


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("L", [1024, 1025, 1535])
def test_outputs_over_the_gate_input(L, io):
    """z and y in one buffer: segments would keep states in rows of y that the gate has yet to be read from."""
    P, N, H, batch = 64, 64, 2, 2
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, 1, batch, L, seed=21)
    a, b = HipLayer(dec, lp, conv_init=conv_init), HipLayer(dec, lp, conv_init=conv_init)
    z = to_dev(tok["z"], io)
    y = torch.empty_like(z)
    _prefill(a, tok, bias, io, L, y, z)
    over = z.clone()
    _prefill(b, tok, bias, io, L, over, over)
    tol = TOL[io]
    assert rel_err(to_host(over), to_host(y)) <= tol
    assert rel_err(to_host(_materialize(b, bias)), to_host(_materialize(a, bias))) <= (1e-4 if io == "bf16" else 1e-5)


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_strong_decay_across_segments(io):
    """Decay of up to e^-30 per token: the summed exponent of a segment is far below the smallest float's."""
    P, N, H, batch, L = 128, 64, 2, 2, 1100
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, 1, batch, L, seed=31)
    lp.A[:] = lp.A * 60.0
    hip, ora = HipLayer(dec, lp), oracle.EagerOracle("scalar", lp.A, lp.D, lp.conv_w, lp.conv_b, lp.h0, io, "none", 1, dt_bias=bias, dt_softplus=True)
    y = torch.empty_like(to_dev(tok["x"], io))
    _prefill(hip, tok, bias, io, L, y, None)
    y_ref, _, _ = ora.verify(tok["x"], tok["dt"], tok["B"], tok["C"])
    ora.commit(np.full(batch, L))
    assert rel_err(to_host(y), y_ref) <= TOL[io] and rel_err(to_host(_materialize(hip, bias)), ora.h) <= TOL[io]


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 130])
def test_every_sequence_of_a_ragged_batch_is_taken_once(batch, io):
    """Workgroups take the sequences in order of length (up to 64 of them) or as they come: equal lengths, empty prompts, more
    sequences than lanes."""
    P, N, H, L = 32, 32, 3, 70
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, 1, batch, L, seed=batch)
    rng = np.random.default_rng(batch)
    lens = rng.choice([0, 1, 5, 32, 33, 69, 70], size=batch).astype(np.int32)
    hip = HipLayer(dec, lp, conv_init=conv_init)
    y = torch.full((batch, L, H * P), 7.0, dtype=torch.bfloat16 if io == "bf16" else torch.float32, device="cuda")
    _prefill(hip, tok, bias, io, L, y, to_dev(tok["z"], io), lens)
    y_h, h_g = to_host(y), to_host(_materialize(hip, bias))
    for b, n in enumerate(int(v) for v in lens):
        ora = oracle.EagerOracle("scalar", lp.A, lp.D, lp.conv_w, lp.conv_b, lp.h0[b:b + 1], io, dec.conv_act, 1, dt_bias=bias, dt_softplus=True,
                                 conv_init=conv_init[b:b + 1])
        if n:
            y_ref, _, _ = ora.verify(tok["x"][b:b + 1, :n], tok["dt"][b:b + 1, :n], tok["B"][b:b + 1, :n], tok["C"][b:b + 1, :n], z=tok["z"][b:b + 1, :n])
            ora.commit([n])
            assert rel_err(y_h[b, :n], y_ref[0]) <= TOL[io], "sequence %d" % b
        assert np.all(y_h[b, n:] == 7.0) and rel_err(h_g[b:b + 1], ora.h) <= TOL[io], "sequence %d" % b
    assert hip.cache.ints()["pos"].tolist() == lens.tolist()


@pytest.mark.parametrize("P,N", SHAPES)
def test_large_state_under_a_decay(P, N):
    """fp32: C h^T is beyond fp32's range, exp(cum) C h^T is not."""
    H, L = 2, 40
    dims = ssmv.make_dims(1, H, P, N, kmax=4, io="f32")
    full = lambda v, *s: torch.full(s, v, device="cuda")
    cache = ssmv.LayerCache.allocate(dims)
    ssmv.ssmv_cache_reset(dims, cache.c, full(1e25, 1, H, P, N), None)
    y = full(7.0, 1, L, H * P)
    ssmv.ssm_prefill_chunked(dims, cache.c, full(1.0, 1, L, H * P), full(0.0, H * P, 4), None, full(40.0, 1, L, H), full(1.0, 1, L, 1, N),
                             full(1e14, 1, L, 1, N), full(-1.0, H), full(0.0, H), L, y)
    want = N * 1e39 * np.exp(-40.0 * (1 + np.arange(L)))
    got = to_host(y)[0]
    # the exponent carries the rounding of 40 t; where exp leaves the normal range, y is zero or nearly
    np.testing.assert_allclose(got[:2], np.repeat(want[:2, None], H * P, 1), rtol=2e-5)
    assert np.all(np.isfinite(got)) and np.all(np.abs(got[3:]) < 1e-6 * want[0])


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("batch,H,L", [(3, 86, 65), (52, 5, 70), (57, 5, 100), (63, 5, 70), (64, 5, 70), (65, 5, 70), (64, 4, 70), (64, 5, 64)])
def test_ragged_batches_in_order_of_length(batch, H, L, io):
    """Up to 64 sequences of more than two chunks, on more than 256 workgroups, are ranked by length: at the edges of that rule
    every sequence gives what it gives in a call of its own."""
    P, N = 32, 32
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, 1, batch, L, seed=batch)
    lens = np.random.default_rng(batch).choice([0, 1, 5, 32, 33, L - 1, L], size=batch).astype(np.int32)

    def run(first, n):
        part = lambda a: a[first:first + n]
        hip = HipLayer(dec.scaled(batch=n), dataclasses.replace(lp, h0=part(lp.h0)), conv_init=part(conv_init))
        y = torch.full((n, L, H * P), 7.0, dtype=torch.bfloat16 if io == "bf16" else torch.float32, device="cuda")
        _prefill(hip, {k: part(v) for k, v in tok.items()}, bias, io, L, y, to_dev(part(tok["z"]), io), part(lens))
        return y, _materialize(hip, bias), hip.cache.ints()

    y, h, ints = run(0, batch)
    assert ints["pos"].tolist() == lens.tolist() and ints["err_flag"] == 0
    for b in range(batch):
        y1, h1, _ = run(b, 1)
        assert torch.equal(y[b:b + 1], y1) and torch.equal(h[b:b + 1], h1), "sequence %d" % b
        assert bool((y[b, lens[b]:] == 7).all())


def _launches(call):
    """Kernel launches of a call: the nodes of a graph it is captured into (and that is not run)."""
    path = next(m.group() for m in (re.search(r"/\S*libamdhip64\S*", line) for line in open("/proc/self/maps")) if m)
    side, graph, n = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True), ctypes.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        graph.capture_begin()
        call()
        graph.capture_end()
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


CUT, UNCUT = 3, 2           # two passes and the launch between them, or one and the bookkeeping


def _launches_of(io, P, N, H, batch, L, lens=None, in_place=False, act="none"):
    dims = ssmv.make_dims(batch, H, P, N, kmax=4, io=io, conv_act=act)
    cache = ssmv.LayerCache.allocate(dims)
    new = lambda *s: torch.zeros(*s, dtype=torch.bfloat16 if io == "bf16" else torch.float32, device="cuda")
    x, y, w, dt, B, C, A = new(batch, L, H * P), new(batch, L, H * P), new(H * P, 4), new(batch, L, H), new(batch, L, 1, N), new(batch, L, 1, N), torch.zeros(H, device="cuda")
    seq_len = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    return _launches(lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=C, A=A, D=A, L=L, y_out=y, z=y if in_place else None,
                                                    seq_len=seq_len))


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_which_prompts_are_cut(io):
    """The prompts of this file that are to be cut are, those that are not to be are not, and lengths of a call's sequences, which the
    device knows, do not matter."""
    for P, N in SHAPES:
        assert _launches_of(io, P, N, 4, 7, 1200) == _launches_of(io, P, N, 4, 7, 1200, lens=[1] * 7) == CUT, (P, N)
        assert _launches_of(io, P, N, 4, 7, 64) == UNCUT
    for L in (1024, 1025, 1535):
        assert _launches_of(io, 64, 64, 2, 2, L) == CUT and _launches_of(io, 64, 64, 2, 2, L, in_place=True) == UNCUT
    assert _launches_of(io, 128, 64, 2, 2, 1100) == CUT
    assert _launches_of(io, 32, 32, 1, 70, 1100) == CUT
    assert _launches_of(io, 128, 64, 80, 4, 1500) == UNCUT            # as many workgroups as fit without
    if io == "bf16":                                                  # few chunks of a small tile: the passes cost more than they save
        assert _launches_of(io, 64, 32, 80, 4, 400) == UNCUT and _launches_of(io, 32, 32, 80, 4, 400) == UNCUT


@pytest.mark.parametrize("P,N,H,batch,L", [(128, 32, 4, 2, 400), (128, 64, 4, 12, 700), (64, 32, 4, 1, 400)])
def test_a_conv_silu_is_counted(P, N, H, batch, L):
    """bf16: a chunk takes longer with it, so that cutting pays earlier."""
    assert _launches_of("bf16", P, N, H, batch, L) == UNCUT and _launches_of("bf16", P, N, H, batch, L, act="silu") == CUT


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_segments_of_more_sequences_than_lanes(io):
    """A ragged batch of more than 64 sequences, cut: workgroups take the sequences as they come."""
    P, N, H, batch, L = 32, 32, 1, 70, 1100
    dec, data, lp, tok, bias, conv_init = _inputs(io, P, N, H, 1, batch, L, seed=41)
    lens = np.random.default_rng(41).choice([0, 1, 31, 64, 65, 200], size=batch).astype(np.int32)
    lens[[3, 40, 69]] = L, 700, L - 1
    hip = HipLayer(dec, lp, conv_init=conv_init)
    y = torch.full((batch, L, H * P), 7.0, dtype=torch.bfloat16 if io == "bf16" else torch.float32, device="cuda")
    _prefill(hip, tok, bias, io, L, y, None, lens)
    y_h, h_g = to_host(y), to_host(_materialize(hip, bias))
    for b, n in enumerate(int(v) for v in lens):
        ora = oracle.EagerOracle("scalar", lp.A, lp.D, lp.conv_w, lp.conv_b, lp.h0[b:b + 1], io, dec.conv_act, 1, dt_bias=bias, dt_softplus=True,
                                 conv_init=conv_init[b:b + 1])
        if n:
            y_ref, _, _ = ora.verify(*(tok[m][b:b + 1, :n] for m in ("x", "dt", "B", "C")))
            ora.commit([n])
            assert rel_err(y_h[b, :n], y_ref[0]) <= TOL[io], "sequence %d" % b
        assert np.all(y_h[b, n:] == 7.0) and rel_err(h_g[b:b + 1], ora.h) <= TOL[io], "sequence %d" % b
    assert hip.cache.ints()["pos"].tolist() == lens.tolist()


# (headdim, dstate, pairs, tokens, whether lengths are given): the ends of the lines within which the bf16 kernel of the large launches
# (csrc/prefill_bf16.hip) cuts a prompt, which the pipelined one would cut into fewer segments or leave whole
OTHER_CUTS = [(32, 32, 112, 3000, False), (32, 32, 448, 3000, False), (32, 32, 112, 1500, True), (32, 32, 256, 1500, True), (32, 32, 80, 2048, True), (32, 32, 384, 2048, True),
              (32, 128, 288, 1500, False), (32, 128, 384, 1500, False), (32, 128, 80, 3000, False), (32, 128, 192, 3000, False), (32, 128, 64, 3000, True),
              (32, 128, 144, 3000, True), (64, 32, 144, 2048, False), (64, 32, 256, 2048, False), (64, 32, 80, 1024, True), (64, 32, 224, 1024, True),
              (128, 32, 48, 1500, False), (128, 32, 176, 1500, False), (128, 32, 80, 1024, True), (128, 32, 144, 1024, True), (128, 32, 32, 1500, True), (128, 32, 208, 1500, True)]


@pytest.mark.parametrize("P,N,pairs,L,lens", OTHER_CUTS)
def test_which_kernel_cuts(P, N, pairs, L, lens):
    """At the ends of a line the other kernel cuts (its first pass: threads of one wave per 32 channels and half of a large state); a token
    less, a pair less or more, lengths not given (or given), or y over the gate, and the pipelined kernel takes the prompt."""
    def first(pairs, L, lens, in_place=False):
        H = 4 if pairs % 4 == 0 else 1
        batch = pairs // H
        dims = ssmv.make_dims(batch, H, P, N, kmax=4, io="bf16")
        cache = ssmv.LayerCache.allocate(dims)
        new = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
        x, y, w, dt, B, C, A = new(batch, L, H * P), new(batch, L, H * P), new(H * P, 4), new(batch, L, H), new(batch, L, 1, N), new(batch, L, 1, N), torch.zeros(H, device="cuda")
        seq_len = torch.full((batch,), L, dtype=torch.int32, device="cuda") if lens else None
        made = launches(lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=C, A=A, D=A, L=L, y_out=y, z=y if in_place else None, seq_len=seq_len))
        return len(made), made[0][1] == (4 * P if N == 128 else 2 * P)

    rule = lambda pairs, L, lens: any((P, N, lens) == (p, n, given) and lo <= pairs <= hi and L >= tokens for p, n, given, tokens, lo, hi in (
        (32, 32, False, 3000, 112, 448), (32, 32, True, 1500, 112, 256), (32, 32, True, 2048, 80, 384), (32, 128, False, 1500, 288, 384), (32, 128, False, 3000, 80, 192),
        (32, 128, True, 3000, 64, 144), (64, 32, False, 2048, 144, 256), (64, 32, True, 1024, 80, 224), (128, 32, False, 1500, 48, 176), (128, 32, True, 1024, 80, 144),
        (128, 32, True, 1500, 32, 208)))
    assert rule(pairs, L, lens) and first(pairs, L, lens) == (CUT, True)
    assert first(pairs, L, lens, in_place=True) == (UNCUT, False)
    for q in ((pairs, L - 1, lens), (pairs - 1, L, lens), (pairs + 1, L, lens), (pairs, L, not lens)):
        assert first(*q)[1] == rule(*q), q


@pytest.mark.parametrize("P,N,pairs,L,lens", OTHER_CUTS[::2])
def test_segments_of_the_other_kernel_against_the_oracle(P, N, pairs, L, lens):
    """A cut prompt behind another one (so that state, ring and conv_head are in the middle of something), then a decoding round; with SiLU,
    gate, softplus and two groups, tiled or row-major slots.  The oracle runs a head of either group in two sequences."""
    H, G, k, io = 4 if pairs % 16 else 16, 2, 4, torch.bfloat16
    batch = pairs // H
    assert H * batch == pairs
    g = torch.Generator(device="cuda").manual_seed(pairs)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    bf, Cx = (lambda t: t.to(io)), H * P
    w, bias, D, dtb = bf(rnd(Cx, 4) / 2), bf(rnd(Cx) * 0.1), rnd(H), torch.rand(H, generator=g, device="cuda") - 0.5
    A = -torch.exp(torch.rand(H, generator=g, device="cuda") * 2.7)
    heads, seqs = [1, H - 1], [0, batch - 1]
    ch = np.concatenate([np.arange(h * P, (h + 1) * P) for h in heads])
    dims = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=k, io="bf16", conv_act="silu", engine="vector" if lens else "auto")
    cache = ssmv.LayerCache.allocate(dims)
    h0, conv0 = rnd(batch, H, P, N) * 0.1, bf(rnd(batch, 3, Cx))
    ssmv.ssmv_cache_reset(dims, cache.c, h0, conv0)
    oras = [oracle.EagerOracle("scalar", to_host(A)[heads], to_host(D)[heads], to_host(w)[ch], to_host(bias)[ch], to_host(h0[b:b + 1])[:, heads], "bf16", "silu", G,
                               conv_init=to_host(conv0[b:b + 1])[:, :, ch], dt_bias=to_host(dtb)[heads], dt_softplus=True) for b in seqs]

    def compare(tok, y, lens, what):
        for ora, b in zip(oras, seqs):
            n = int(lens[b])
            f = lambda t, sel: to_host(t[b:b + 1, :n])[:, :, sel]
            y_ref, _, _ = ora.verify(f(tok["x"], ch), f(tok["dt"], heads), to_host(tok["B"][b:b + 1, :n]), to_host(tok["C"][b:b + 1, :n]), z=f(tok["z"], ch))
            ora.commit([n])
            assert rel_err(f(y, ch), y_ref) <= TOL["bf16"], "%s, sequence %d" % (what, b)
            assert bool((y[b, n:] == 7).all()), "%s, sequence %d: outputs behind its length" % (what, b)

    for n, what in ((37, "short prompt"), (L, "cut prompt"), (k, "decoding")):
        tok = dict(x=bf(rnd(batch, n, Cx)), dt=bf(rnd(batch, n, H) - 4), B=bf(rnd(batch, n, G, N) / N ** 0.5), C=bf(rnd(batch, n, G, N) / N ** 0.5), z=bf(rnd(batch, n, Cx)))
        y, given, seq_len = torch.full_like(tok["x"], 7.0), torch.full((batch,), n, dtype=torch.int32), None
        common = dict(x_raw=tok["x"], conv_wgt=w, conv_bias=bias, dt=tok["dt"], dt_bias=dtb, dt_softplus=True, Bm=tok["B"], Cm=tok["C"], z=tok["z"], A=A, D=D, y_out=y)
        if what == "decoding":
            ssmv.ssm_block_multistep(dims, cache.c, k=k, **common)
        else:
            if lens:
                given = torch.randint(1, n + 1, (batch,), generator=torch.Generator().manual_seed(n), dtype=torch.int32)
                given[0], given[-1] = n, n - 33
                seq_len = given.cuda()
            run = lambda: ssmv.ssm_prefill_block(dims, cache.c, L=n, seq_len=seq_len, **common)
            if what == "cut prompt":
                made = launches(run)
                assert len(made) == CUT and made[0][1] == (4 * P if N == 128 else 2 * P)
            run()
        compare(tok, y, given, what)
        if what == "cut prompt":
            h = torch.empty_like(h0)
            ssmv.ssmv_materialize_block(dims, cache.c, A, dtb, True, h)
            for ora, b in zip(oras, seqs):
                assert rel_err(to_host(h[b:b + 1])[:, heads], ora.h) <= TOL["bf16"], "sequence %d: state" % b
    ssmv.ssmv_check(cache.c)
