"""fp32 prefill launches of every size: which of the two kernels a call runs, whole, in parts or cut (csrc/prefill.hip: plan_f32), and both of
them against the oracle where the other test files' small calls do not take them (csrc/prefill.hip, csrc/prefill_f32_pipe.hip)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_15237_amd as ssmv

from _harness import TOL, launches, rel_err, to_host

pytestmark = pytest.mark.gpu

PIPE, OTHER = 1, 0


def first_launch(P, N, pairs, kernel, parts, segments):
    """Launches of a call, and workgroups and threads of its first one."""
    def threads(P):                                                    # of the pipelined kernel: consumers, three weight waves, the decay wave, four conv waves
        tiles, shares = P // 32, min(max(N // 32, 1), 4 // (P // 32))
        return 64 * (tiles * shares + 8)
    return 3 if segments else 2, (pairs * parts * max(1, segments - 1), threads(P // parts) if kernel == PIPE else 256)


def made(run):
    launched = launches(run)
    return len(launched), launched[0]


# (headdim, dstate, heads, batch, tokens, whether lengths are given, kernel, parts, segments): both sides of a line of every tile
LINES = [
    (32, 32, 4, 64, 33, False, PIPE, 1, 0), (32, 32, 4, 65, 33, False, OTHER, 1, 0), (32, 32, 4, 83, 33, True, PIPE, 1, 0),
    (32, 32, 4, 84, 33, True, OTHER, 1, 0), (32, 64, 4, 64, 33, False, PIPE, 1, 0), (32, 64, 4, 65, 33, False, OTHER, 1, 0),
    (32, 64, 4, 101, 33, True, PIPE, 1, 0), (32, 64, 4, 102, 33, True, OTHER, 1, 0), (32, 128, 4, 192, 33, False, PIPE, 1, 0),
    (32, 128, 4, 193, 33, False, OTHER, 1, 0), (32, 128, 4, 117, 33, True, PIPE, 1, 0), (32, 128, 4, 118, 33, True, OTHER, 1, 0),
    (64, 32, 4, 64, 33, False, PIPE, 1, 0), (64, 32, 4, 65, 33, False, OTHER, 1, 0), (64, 32, 4, 90, 33, True, PIPE, 1, 0),
    (64, 32, 4, 91, 33, True, OTHER, 1, 0), (64, 64, 4, 128, 33, False, PIPE, 1, 0), (64, 64, 4, 129, 33, False, OTHER, 1, 0),
    (64, 64, 4, 118, 33, True, PIPE, 1, 0), (64, 64, 4, 119, 33, True, OTHER, 1, 0), (64, 128, 4, 64, 33, False, PIPE, 1, 0),
    (64, 128, 4, 65, 33, False, OTHER, 1, 0), (64, 128, 4, 111, 33, True, PIPE, 1, 0), (64, 128, 4, 112, 33, True, OTHER, 1, 0),
    (128, 32, 4, 64, 33, False, PIPE, 1, 0), (128, 32, 4, 65, 33, False, OTHER, 1, 0), (128, 32, 4, 94, 33, True, PIPE, 1, 0),
    (128, 32, 4, 95, 33, True, OTHER, 1, 0), (128, 64, 4, 117, 33, True, PIPE, 1, 0), (128, 64, 4, 118, 33, True, OTHER, 1, 0),
    (128, 128, 4, 64, 65, False, OTHER, 1, 0), (128, 128, 4, 65, 65, False, PIPE, 2, 0), (128, 128, 4, 53, 33, True, PIPE, 2, 0),
    (128, 128, 4, 54, 33, True, OTHER, 1, 0),
    # the sizes whose times stand beside the plan
    (128, 64, 32, 4, 1021, False, PIPE, 2, 0), (128, 64, 32, 32, 2048, False, PIPE, 1, 0), (128, 128, 32, 16, 512, False, OTHER, 1, 0),
    # given lengths, which may all be the longest: as many parts as lose little there
    (64, 32, 7, 22, 2324, True, PIPE, 1, 0), (64, 32, 7, 22, 2324, False, OTHER, 1, 5), (32, 32, 64, 16, 800, True, OTHER, 1, 0),
    (32, 64, 64, 16, 200, True, OTHER, 1, 0), (128, 64, 5, 17, 1352, True, PIPE, 1, 4), (32, 32, 57, 10, 340, True, PIPE, 1, 0),
    (128, 128, 57, 9, 200, True, OTHER, 1, 0)]


@pytest.mark.parametrize("P,N,H,batch,L,lens,kernel,parts,segments", LINES)
def test_which_kernel_a_call_runs(P, N, H, batch, L, lens, kernel, parts, segments):
    new = lambda *s: torch.zeros(*s, device="cuda")
    dims = ssmv.make_dims(batch, H, P, N, kmax=4, io="f32")
    cache = ssmv.LayerCache.allocate(dims)
    x, y, w, dt, B, A = new(batch, L, H * P), new(batch, L, H * P), new(H * P, 4), new(batch, L, H), new(batch, L, 1, N), new(H)
    seq_len = torch.full((batch,), L, dtype=torch.int32, device="cuda") if lens else None
    run = lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=B, A=A, D=A, L=L, y_out=y, seq_len=seq_len)
    assert made(run) == first_launch(P, N, H * batch, kernel, parts, segments)


def against_the_oracle(P, N, H, batch, L, mode, expected, seed=0):
    """Two prompts one after the other (the second continues the ring and the state of the first), then a decoding round.  mode "plain":
    nothing but the recurrence; "lens": given lengths; "block": given lengths, SiLU, gate (outputs over it, or beside it where the prompt is
    cut), softplus, conv bias, row-major slots.  The oracle runs two heads of either group in three sequences."""
    G, k, block = 2 if H % 2 == 0 else 1, 4, mode == "block"
    g = torch.Generator(device="cuda").manual_seed(P + N + L + seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    Cx = H * P
    w, bias, D, dtb = rnd(Cx, 4) / 2, rnd(Cx) * 0.1 if block else None, rnd(H), torch.rand(H, generator=g, device="cuda") - 0.5
    A, act = -torch.exp(torch.rand(H, generator=g, device="cuda") * 2.7), "silu" if block else "none"
    per = H // G
    heads, seqs = sorted({0, per - 1, H - per, H - 1}), sorted({0, batch // 2, batch - 1})     # as many of either group
    ch = np.concatenate([np.arange(h * P, (h + 1) * P) for h in heads])
    dims = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=k, io="f32", conv_act=act, engine="vector" if block else "auto")
    cache = ssmv.LayerCache.allocate(dims)
    h0, conv0 = rnd(batch, H, P, N) * 0.1, rnd(batch, 3, Cx)
    ssmv.ssmv_cache_reset(dims, cache.c, h0, conv0)
    oras = [oracle.EagerOracle("scalar", to_host(A)[heads], to_host(D)[heads], to_host(w)[ch], to_host(bias)[ch] if block else None, to_host(h0[b:b + 1])[:, heads], "f32", act, G,
                               conv_init=to_host(conv0[b:b + 1])[:, :, ch], dt_bias=to_host(dtb)[heads] if block else None, dt_softplus=block) for b in seqs]
    in_place = block and not expected[2]
    # of the other kernel a token's weight in the state is exp of the difference of two prefix sums over a chunk, each with the rounding of its last two
    # additions at its own size, 2^-24 of it, before all: 4 x 2^-24 x |A| sum dt of the weight's value on top of what a sum has
    steps = lambda dt: torch.nn.functional.softplus(dt + dtb) if block else dt
    bound = lambda b, tok: TOL["f32"] + (0.0 if expected[0] == PIPE else 2.0 ** -22 * float(torch.stack([(steps(c[b]) * -A).sum(0)[heads] for c in tok["dt"].split(32, 1)]).max()))
    for what in ("first prompt", "second prompt", "decoding"):
        n = k if what == "decoding" else L
        tok = dict(x=rnd(batch, n, Cx), dt=rnd(batch, n, H) - 4 if block else torch.nn.functional.softplus(rnd(batch, n, H) - 4), B=rnd(batch, n, G, N) / N ** 0.5,
                   C=rnd(batch, n, G, N) / N ** 0.5, z=rnd(batch, n, Cx) if block else None)
        lens = torch.full((batch,), n, dtype=torch.int32)
        if mode != "plain" and what != "decoding":
            lens = torch.randint(0, n + 1, (batch,), generator=torch.Generator().manual_seed(L + len(what)), dtype=torch.int32)
            lens[seqs[-1]] = n
        y = tok["z"].clone() if in_place else torch.full_like(tok["x"], 7.0)
        kept = y.clone()
        common = dict(x_raw=tok["x"], conv_wgt=w, conv_bias=bias, dt=tok["dt"], dt_bias=dtb if block else None, dt_softplus=block, Bm=tok["B"], Cm=tok["C"],
                      z=y if in_place else tok["z"], A=A, D=D, y_out=y)
        if what == "decoding":
            ssmv.ssm_block_multistep(dims, cache.c, k=k, **dict(common, z=tok["z"]))
        else:
            lens_dev = lens.cuda() if mode != "plain" else None
            run = lambda: ssmv.ssm_prefill_block(dims, cache.c, L=n, seq_len=lens_dev, **common)
            assert made(run) == first_launch(P, N, H * batch, *expected), what
            run()
        for ora, b in zip(oras, seqs):
            m = int(lens[b])
            if m:
                f = lambda t, sel: to_host(t[b:b + 1, :m])[:, :, sel]
                y_ref, _, _ = ora.verify(f(tok["x"], ch), f(tok["dt"], heads), to_host(tok["B"][b:b + 1, :m]), to_host(tok["C"][b:b + 1, :m]), z=f(tok["z"], ch) if block else None)
                ora.commit([m])
                assert rel_err(f(y, ch), y_ref) <= TOL["f32"], "%s, sequence %d" % (what, b)
            assert torch.equal(y[b, m:], kept[b, m:]), "%s, sequence %d: outputs behind its length" % (what, b)
        if what != "decoding":
            h = torch.empty_like(h0)
            ssmv.ssmv_materialize_block(dims, cache.c, A, dtb if block else None, block, h)
            for ora, b in zip(oras, seqs):
                assert rel_err(to_host(h[b:b + 1])[:, heads], ora.h) <= bound(b, tok), "%s, sequence %d: state" % (what, b)
    ssmv.ssmv_check(cache.c)


# (headdim, dstate, heads, batch, mode, lengths): more pairs than the pipelined kernel is the faster for, where there are such (of one
# length 64 x 64, 64 x 128, 128 x 64 and 32 x 128 up to a few chunks)
LARGE = [
    (32, 32, 6, 43, "plain", (1, 31, 32, 33, 65, 161)), (32, 32, 12, 43, "lens", (1, 33, 161)), (32, 32, 12, 43, "block", (1, 31, 32, 33, 65, 161)),
    (32, 64, 12, 43, "plain", (1, 31, 32, 33, 65, 161)), (32, 64, 62, 12, "lens", (1, 33, 161)), (32, 64, 62, 12, "block", (1, 31, 32, 33, 65, 161)),
    (32, 128, 22, 35, "plain", (1, 31, 32, 33)), (32, 128, 28, 32, "lens", (1, 33, 161)), (32, 128, 28, 32, "block", (1, 31, 32, 33, 65, 161)),
    (64, 32, 6, 43, "plain", (1, 31, 32, 33, 65, 161)), (64, 32, 62, 10, "lens", (1, 33, 161)), (64, 32, 62, 10, "block", (1, 31, 32, 33, 65, 161)),
    (64, 64, 12, 43, "plain", (1, 31, 32, 33, 65, 97)), (64, 64, 62, 15, "lens", (1, 33, 161)), (64, 64, 62, 15, "block", (1, 31, 32, 33, 65, 161)),
    (64, 128, 10, 39, "plain", (1, 31, 32, 33, 65)), (64, 128, 58, 11, "lens", (1, 33, 161)), (64, 128, 58, 11, "block", (1, 31, 32, 33, 65, 161)),
    (128, 32, 6, 43, "plain", (1, 31, 32, 33, 65, 161)), (128, 32, 44, 14, "lens", (1, 33, 161)), (128, 32, 44, 14, "block", (1, 31, 32, 33, 65, 161)),
    (128, 64, 10, 39, "plain", (1, 31, 32, 33)), (128, 64, 48, 14, "lens", (1, 33, 161)), (128, 64, 48, 14, "block", (1, 31, 32, 33, 65, 161)),
    (128, 128, 10, 39, "plain", (1, 31, 32, 33, 65, 161)), (128, 128, 62, 7, "lens", (1, 33, 161)), (128, 128, 62, 7, "block", (1, 31, 32, 33, 65, 161))]


@pytest.mark.parametrize("P,N,H,batch,mode,lengths", LARGE)
def test_large_launches_of_the_other_kernel(P, N, H, batch, mode, lengths):
    for L in lengths:
        against_the_oracle(P, N, H, batch, L, mode, (OTHER, 1, 0))


# (headdim, dstate, heads, batch, parts): the pipelined kernel over five and more chunks, undivided on every tile, and in parts
PIPED = [(32, 32, 16, 16, 1), (32, 64, 16, 16, 1), (32, 128, 16, 16, 1), (64, 32, 16, 16, 1), (64, 64, 16, 16, 1), (64, 128, 16, 16, 1), (128, 32, 16, 16, 1), (128, 64, 16, 16, 1),
         (64, 32, 8, 12, 2), (64, 64, 8, 12, 2), (64, 128, 8, 12, 2), (128, 32, 8, 12, 2), (128, 64, 8, 12, 2), (128, 128, 8, 16, 2), (128, 32, 4, 10, 4), (128, 64, 4, 10, 4), (128, 128, 4, 10, 4)]


@pytest.mark.parametrize("mode", ["plain", "block"])
@pytest.mark.parametrize("P,N,H,batch,parts", PIPED)
def test_pipelined_kernel_over_many_chunks(P, N, H, batch, parts, mode):
    against_the_oracle(P, N, H, batch, 175, mode, (PIPE, parts, 0))


# (headdim, dstate, heads, batch, tokens, mode, kernel, parts, segments): every instantiation that takes a segment
CUTS = [
    (32, 32, 6, 1, 2755, "plain", OTHER, 1, 44), (32, 32, 6, 1, 4169, "block", OTHER, 1, 66), (32, 64, 12, 2, 1745, "plain", OTHER, 1, 19),
    (32, 64, 8, 2, 3563, "block", OTHER, 1, 38), (64, 32, 6, 1, 1947, "plain", OTHER, 1, 31), (64, 32, 6, 1, 4169, "block", OTHER, 1, 66),
    (64, 64, 6, 3, 2048, "plain", OTHER, 1, 22), (64, 64, 8, 2, 3563, "block", OTHER, 1, 38), (64, 128, 12, 2, 3260, "plain", OTHER, 1, 21),
    (128, 32, 2, 1, 4169, "plain", OTHER, 1, 66), (128, 32, 6, 1, 2957, "block", OTHER, 1, 47), (128, 64, 12, 1, 3462, "plain", OTHER, 1, 37),
    (128, 128, 12, 1, 4068, "plain", OTHER, 1, 22), (128, 128, 6, 3, 4169, "block", OTHER, 1, 27),
    (32, 32, 2, 1, 331, "plain", PIPE, 1, 6), (32, 32, 2, 1, 331, "block", PIPE, 1, 6), (32, 64, 2, 1, 331, "plain", PIPE, 1, 4), (32, 64, 2, 1, 331, "block", PIPE, 1, 4),
    (32, 128, 2, 1, 432, "plain", PIPE, 1, 3), (32, 128, 2, 1, 432, "block", PIPE, 1, 3), (64, 32, 2, 1, 4169, "plain", PIPE, 1, 66), (64, 32, 2, 1, 4169, "block", PIPE, 1, 66),
    (64, 32, 2, 1, 331, "plain", PIPE, 2, 6), (64, 64, 14, 2, 331, "plain", PIPE, 1, 4), (64, 64, 14, 2, 331, "block", PIPE, 1, 4), (64, 64, 2, 1, 331, "block", PIPE, 2, 4),
    (64, 128, 8, 1, 3563, "plain", PIPE, 1, 23), (64, 128, 8, 1, 3563, "block", PIPE, 1, 23), (64, 128, 2, 1, 432, "block", PIPE, 2, 3), (128, 32, 6, 1, 2149, "plain", PIPE, 1, 34),
    (128, 32, 8, 1, 1240, "block", PIPE, 1, 20), (128, 32, 6, 1, 735, "plain", PIPE, 2, 12), (128, 32, 2, 1, 331, "block", PIPE, 4, 6), (128, 64, 12, 1, 1745, "plain", PIPE, 1, 19),
    (128, 64, 12, 1, 1745, "block", PIPE, 1, 19), (128, 64, 14, 1, 331, "plain", PIPE, 2, 4), (128, 64, 2, 1, 331, "block", PIPE, 4, 4), (128, 128, 4, 1, 3563, "plain", PIPE, 2, 23),
    (128, 128, 22, 1, 533, "block", PIPE, 2, 4), (128, 128, 2, 1, 432, "block", PIPE, 4, 3)]


@pytest.mark.parametrize("P,N,H,batch,L,mode,kernel,parts,segments", CUTS)
def test_cut_prompts_against_the_oracle(P, N, H, batch, L, mode, kernel, parts, segments):
    against_the_oracle(P, N, H, batch, L, mode, (kernel, parts, segments))


@pytest.mark.parametrize("P,N,H,batch", [(32, 32, 6, 43), (32, 64, 12, 43), (64, 32, 6, 43), (64, 64, 12, 43), (64, 128, 10, 39), (128, 32, 6, 43), (128, 64, 10, 39), (128, 128, 10, 39),
                                         (32, 128, 22, 35)])
def test_large_state_under_a_decay(P, N, H, batch):
    """The other kernel, where C h^T is beyond fp32's range and exp(cum) C h^T is not; then a decay of up to e^-30 a token."""
    L = 33
    dims = ssmv.make_dims(batch, H, P, N, kmax=4, io="f32")
    full = lambda v, *s: torch.full(s, v, device="cuda")
    cache = ssmv.LayerCache.allocate(dims)
    ssmv.ssmv_cache_reset(dims, cache.c, full(1e25, batch, H, P, N), None)
    x, w, y, A, D = full(1.0, batch, L, H * P), full(0.0, H * P, 4), full(7.0, batch, L, H * P), full(-1.0, H), full(0.0, H)
    dt, B, C = full(40.0, batch, L, H), full(1.0, batch, L, 1, N), full(1e14, batch, L, 1, N)
    run = lambda: ssmv.ssm_prefill_chunked(dims, cache.c, x, w, None, dt, B, C, A, D, L, y)
    assert made(run) == first_launch(P, N, H * batch, OTHER, 1, 0)
    run()
    want, got = N * 1e39 * np.exp(-40.0 * (1 + np.arange(L))), y.double().cpu().numpy()
    np.testing.assert_allclose(got[:, :2], np.broadcast_to(want[None, :2, None], (batch, 2, H * P)), rtol=2e-5)      # the exponent carries the rounding of 40 t
    assert np.all(np.isfinite(got)) and np.all(np.abs(got[:, 3:]) < 1e-6 * want[0])
    g = torch.Generator(device="cuda").manual_seed(P + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    h0, x, B, C, A, w = rnd(batch, H, P, N), rnd(batch, L, H * P), rnd(batch, L, 1, N) / N ** 0.5, rnd(batch, L, 1, N) / N ** 0.5, -30.0 * torch.rand(H, generator=g, device="cuda"), rnd(H * P, 4)
    dt = torch.rand(batch, L, H, generator=g, device="cuda")
    ssmv.ssmv_cache_reset(dims, cache.c, h0, None)
    ssmv.ssm_prefill_chunked(dims, cache.c, x, w, None, dt, B, C, A, D, L, y)
    h = torch.empty_like(h0)
    ssmv.ssmv_materialize(dims, cache.c, A, h)
    # a weight is exp of the difference of two prefix sums over a chunk, each of which has the rounding of its last two additions at its own size,
    # 2^-24 of it, before all: at most 4 x 2^-24 x |A| sum dt of the weight's value on top of what a call without such decays may have
    for b in (0, batch - 1):
        for hd in (0, 1, H - 1):
            ch, c = slice(hd * P, (hd + 1) * P), slice(hd, hd + 1)
            ora = oracle.EagerOracle("scalar", to_host(A)[c], to_host(D)[c], to_host(w)[ch], None, to_host(h0[b:b + 1])[:, c], "f32", "none", 1)
            y_ref, _, _ = ora.verify(to_host(x[b:b + 1])[:, :, ch], to_host(dt[b:b + 1])[:, :, c], to_host(B[b:b + 1]), to_host(C[b:b + 1]))
            ora.commit([L])
            bound = TOL["f32"] + 2.0 ** -22 * float(-A[hd] * dt[b, :32, hd].sum())
            assert rel_err(to_host(y[b:b + 1])[:, :, ch], y_ref) <= bound and rel_err(to_host(h[b:b + 1])[:, c], ora.h) <= bound, "sequence %d, head %d" % (b, hd)
