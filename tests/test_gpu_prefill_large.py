"""bf16 prefill launches of more (sequence, head) pairs than fit the chip at once: which kernel a call runs, and both of them against
the oracle there (csrc/prefill_bf16.hip, csrc/prefill_pipe.hip)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_15237_amd as ssmv

from _harness import TOL, launches, rel_err, to_host

pytestmark = pytest.mark.gpu


def _threads(P, N):
    """Threads of a workgroup of the pipelined kernel and of the other one."""
    split = 2 if N >= 128 and P <= 64 else 1
    return 64 * (P // 32 * split + (4 if N >= 64 else 2) + P // 32), 2 * P * split


def _prefill_launches(P, N, pairs, L, lens=False):
    H = 4 if pairs % 4 == 0 else 1
    batch = pairs // H
    new = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    dims = ssmv.make_dims(batch, H, P, N, kmax=4, io="bf16")
    cache = ssmv.LayerCache.allocate(dims)
    x, y, w, dt, B, C, A = new(batch, L, H * P), new(batch, L, H * P), new(H * P, 4), new(batch, L, H), new(batch, L, 1, N), new(batch, L, 1, N), torch.zeros(H, device="cuda")
    seq_len = torch.full((batch,), L, dtype=torch.int32, device="cuda") if lens else None
    return launches(lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=C, A=A, D=A, L=L, y_out=y, seq_len=seq_len))


PIPE, OTHER = 0, 1


@pytest.mark.parametrize("P,N,pairs,L,lens,kernel", [
    # a second round of workgroups, which short prompts do not give back
    (64, 64, 512, 1, False, PIPE), (64, 64, 516, 1, False, OTHER), (64, 64, 768, 159, False, OTHER), (64, 64, 768, 160, False, PIPE),
    (64, 64, 772, 1023, False, OTHER), (64, 64, 1024, 1023, False, OTHER), (64, 64, 1024, 1024, False, PIPE), (64, 64, 1028, 64, False, OTHER),
    (64, 64, 1028, 65, False, PIPE), (64, 64, 512, 64, True, PIPE), (64, 64, 768, 159, True, OTHER), (64, 64, 768, 160, True, PIPE),
    (64, 64, 1024, 399, True, OTHER), (64, 64, 1024, 400, True, PIPE), (64, 64, 1280, 699, True, OTHER), (64, 64, 1280, 700, True, PIPE),
    (32, 64, 512, 1, False, PIPE), (32, 64, 516, 127, False, OTHER), (32, 64, 768, 127, True, OTHER), (32, 64, 768, 128, False, PIPE), (32, 64, 772, 200, False, OTHER),
    (32, 128, 256, 1, False, PIPE), (32, 128, 260, 127, False, OTHER), (32, 128, 512, 128, False, PIPE), (32, 128, 516, 200, False, OTHER),
    # launches that one round holds, and lines between the kernels at any length
    (32, 32, 768, 1, False, PIPE), (32, 32, 772, 300, False, OTHER), (64, 32, 512, 1, False, PIPE), (64, 32, 516, 300, False, OTHER),
    (64, 128, 256, 1, False, PIPE), (64, 128, 260, 64, False, OTHER), (128, 32, 256, 1, False, PIPE), (128, 32, 260, 64, False, OTHER),
    (128, 64, 256, 1, False, PIPE), (128, 64, 260, 64, False, OTHER), (128, 128, 1024, 1, False, PIPE),
    # prompts of different lengths: from 512 tokens on, up to twice as many
    (128, 64, 512, 511, True, OTHER), (128, 64, 512, 512, True, PIPE), (128, 64, 516, 512, True, OTHER), (64, 128, 512, 512, True, PIPE), (64, 128, 512, 511, True, OTHER),
    (64, 32, 768, 512, True, PIPE), (64, 32, 772, 512, True, OTHER), (32, 64, 1024, 512, True, PIPE), (32, 64, 1024, 511, True, OTHER), (32, 32, 1024, 512, True, PIPE),
    (32, 32, 1028, 512, True, OTHER), (32, 128, 768, 512, True, PIPE), (32, 128, 772, 512, True, OTHER),
])
def test_which_kernel_a_call_runs(P, N, pairs, L, lens, kernel):
    main = _prefill_launches(P, N, pairs, L, lens)[0]
    assert main == (pairs, _threads(P, N)[kernel])


# (headdim, dstate, heads, batch): one step or a few past the lines, at any length up to 300 tokens
LARGE = [(128, 64, 34, 8), (128, 32, 34, 8), (64, 128, 34, 8), (64, 64, 56, 16), (64, 32, 34, 16), (32, 64, 60, 13), (32, 32, 60, 13), (32, 128, 34, 16)]


@pytest.mark.parametrize("block", [False, True], ids=["plain", "block"])
@pytest.mark.parametrize("P,N,H,batch", LARGE)
def test_large_launches_against_the_oracle(P, N, H, batch, block):
    """Two groups of B and C, two prompts one after the other (the second continues the ring and the state of the first), then a
    decoding round, at lengths around a chunk and at 300 tokens.  block: SiLU, gate, softplus, conv bias, row-major slots, and lengths
    that differ; plain: none of it, tiled slots where the verify kernel takes the shape.  The oracle runs two heads of either group in three sequences."""
    G, io, k = 2, torch.bfloat16, 4
    g = torch.Generator(device="cuda").manual_seed(P + N + block)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    bf = lambda t: t.to(io)
    Cx = H * P
    w, bias, D, dtb = bf(rnd(Cx, 4) / 2), bf(rnd(Cx) * 0.1) if block else None, rnd(H), torch.rand(H, generator=g, device="cuda") - 0.5
    A = -torch.exp(torch.rand(H, generator=g, device="cuda") * 2.7)
    heads, seqs = [0, H // 2 - 1, H // 2, H - 1], [0, 1, batch - 1]
    ch = np.concatenate([np.arange(h * P, (h + 1) * P) for h in heads])
    act = "silu" if block else "none"
    dims = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=k, io="bf16", conv_act=act, engine="vector" if block else "auto")
    host = lambda t: to_host(t)
    tokens = lambda n: dict(x=bf(rnd(batch, n, Cx)), dt=bf(rnd(batch, n, H) - 4 if block else torch.nn.functional.softplus(rnd(batch, n, H) - 4)),
                            B=bf(rnd(batch, n, G, N) / N ** 0.5), C=bf(rnd(batch, n, G, N) / N ** 0.5), z=bf(rnd(batch, n, Cx)) if block else None)
    for L in (1, 3, 31, 32, 33, 64, 65, 300):
        h0, conv0 = rnd(batch, H, P, N) * 0.1, bf(rnd(batch, 3, Cx))
        cache = ssmv.LayerCache.allocate(dims)
        ssmv.ssmv_cache_reset(dims, cache.c, h0, conv0)
        oras = [oracle.EagerOracle("scalar", host(A)[heads], host(D)[heads], host(w)[ch], host(bias)[ch] if block else None, host(h0[b:b + 1])[:, heads], "bf16", act, G,
                                   conv_init=host(conv0[b:b + 1])[:, :, ch], dt_bias=host(dtb)[heads] if block else None, dt_softplus=block) for b in seqs]

        def against_oracle(tok, y, lens, what):
            for ora, b, n in zip(oras, seqs, lens):
                if n:
                    f = lambda t, sel: host(t[b:b + 1, :n])[:, :, sel]
                    y_ref, _, _ = ora.verify(f(tok["x"], ch), f(tok["dt"], heads), host(tok["B"][b:b + 1, :n]), host(tok["C"][b:b + 1, :n]), z=f(tok["z"], ch) if block else None)
                    ora.commit([n])
                    assert rel_err(f(y, ch), y_ref) <= TOL["bf16"], "L = %d, %s, sequence %d" % (L, what, b)
                assert bool((y[b, n:] == 7).all()), "L = %d, %s, sequence %d: outputs behind its length" % (L, what, b)

        for what in ("first prompt", "second prompt"):
            tok = tokens(L)
            lens = torch.randint(0, L + 1, (batch,), generator=torch.Generator().manual_seed(L), dtype=torch.int32) if block else torch.full((batch,), L, dtype=torch.int32)
            if block:
                lens[1] = L
            y = torch.full_like(tok["x"], 7.0)
            run = lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=tok["x"], conv_wgt=w, conv_bias=bias, dt=tok["dt"], dt_bias=dtb if block else None, dt_softplus=block,
                                                 Bm=tok["B"], Cm=tok["C"], z=tok["z"], A=A, D=D, L=L, y_out=y, seq_len=lens_dev)
            lens_dev = lens.cuda() if block else None
            assert launches(run)[0] == (H * batch, _threads(P, N)[OTHER])
            run()
            against_oracle(tok, y, [int(lens[b]) for b in seqs], what)
            h = torch.empty_like(h0)
            ssmv.ssmv_materialize_block(dims, cache.c, A, dtb if block else None, block, h)
            for ora, b in zip(oras, seqs):
                assert rel_err(host(h[b:b + 1])[:, heads], ora.h) <= TOL["bf16"], "L = %d, %s, sequence %d: state" % (L, what, b)
        tok = tokens(k)
        y = torch.full_like(tok["x"], 7.0)
        ssmv.ssm_block_multistep(dims, cache.c, x_raw=tok["x"], conv_wgt=w, conv_bias=bias, dt=tok["dt"], dt_bias=dtb if block else None, dt_softplus=block, Bm=tok["B"],
                                 Cm=tok["C"], z=tok["z"], A=A, D=D, k=k, y_out=y)
        against_oracle(tok, y, [k] * len(seqs), "decoding")
        ssmv.ssmv_check(cache.c)


# (headdim, dstate, heads, batch, tokens, whether lengths differ, kernel)
@pytest.mark.parametrize("P,N,H,batch,L,lens,kernel", [
    (128, 64, 32, 32, 2048, False, OTHER),                             # the bench's launch
    # the pipelined kernel in more than one round: prompts of different lengths, and tiles that it takes at any count
    (128, 64, 32, 16, 530, True, PIPE), (128, 32, 32, 16, 530, True, PIPE), (64, 128, 32, 16, 530, True, PIPE), (64, 32, 48, 16, 530, True, PIPE),
    (32, 64, 64, 16, 530, True, PIPE), (32, 32, 64, 16, 530, True, PIPE), (32, 128, 48, 16, 530, True, PIPE), (64, 64, 80, 16, 710, True, PIPE),
    (64, 64, 64, 20, 100, False, PIPE), (128, 128, 34, 16, 100, False, PIPE)])
def test_more_rounds_and_long_prompts_against_the_oracle(P, N, H, batch, L, lens, kernel):
    G, io = 2, torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(L + P + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    bf, Cx = (lambda t: t.to(io)), H * P
    w, D, A = bf(rnd(Cx, 4) / 2), rnd(H), -torch.exp(torch.rand(H, generator=g, device="cuda") * 2.7)
    x, dt = bf(rnd(batch, L, Cx)), bf(torch.nn.functional.softplus(rnd(batch, L, H) - 4))
    B, C = bf(rnd(batch, L, G, N) / N ** 0.5), bf(rnd(batch, L, G, N) / N ** 0.5)
    h0 = rnd(batch, H, P, N) * 0.1
    dims = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=4, io="bf16")
    cache = ssmv.LayerCache.allocate(dims)
    ssmv.ssmv_cache_reset(dims, cache.c, h0, None)
    given = torch.full((batch,), L, dtype=torch.int32)
    if lens:
        given = torch.randint(0, L + 1, (batch,), generator=torch.Generator().manual_seed(L), dtype=torch.int32)
        given[3] = L
    given_dev, y = given.cuda() if lens else None, torch.full_like(x, 7.0)
    run = lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=C, A=A, D=D, L=L, y_out=y, seq_len=given_dev)
    assert launches(run)[0] == (H * batch, _threads(P, N)[kernel])
    run()
    h = torch.empty_like(h0)
    ssmv.ssmv_materialize(dims, cache.c, A, h)
    ssmv.ssmv_check(cache.c)
    heads = [0, H // 2 - 1, H // 2, H - 1]
    ch = np.concatenate([np.arange(hd * P, (hd + 1) * P) for hd in heads])
    for b in (3, batch - 1):
        n = int(given[b])
        ora = oracle.EagerOracle("scalar", to_host(A)[heads], to_host(D)[heads], to_host(w)[ch], None, to_host(h0[b:b + 1])[:, heads], "bf16", "none", G)
        f = lambda t, sel: to_host(t[b:b + 1, :n])[:, :, sel]
        y_ref, _, _ = ora.verify(f(x, ch), f(dt, heads), to_host(B[b:b + 1, :n]), to_host(C[b:b + 1, :n]))
        ora.commit([n])
        assert rel_err(f(y, ch), y_ref) <= TOL["bf16"] and bool((y[b, n:] == 7).all()), "sequence %d" % b
        assert rel_err(to_host(h[b:b + 1])[:, heads], ora.h) <= TOL["bf16"], "sequence %d: state" % b


@pytest.mark.parametrize("P,N,H,batch", [(128, 64, 34, 8), (64, 128, 34, 8), (64, 64, 56, 16)])
def test_large_launches_with_outputs_over_the_gate_input(P, N, H, batch):
    """y in z's buffer gives what it gives in one of its own, bit for bit."""
    L, io = 100, torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(P * N)
    bf = lambda *s: torch.randn(*s, generator=g, device="cuda").to(io)
    x, z, dt = bf(batch, L, H * P), bf(batch, L, H * P), torch.nn.functional.softplus(bf(batch, L, H) - 4)
    B, C, w, A = bf(batch, L, 1, N), bf(batch, L, 1, N), bf(H * P, 4), -torch.rand(H, generator=g, device="cuda")
    dims = ssmv.make_dims(batch, H, P, N, kmax=4, io="bf16")
    out = []
    for y in (torch.empty_like(z), z.clone()):
        gate = z if not out else y
        cache = ssmv.LayerCache.allocate(dims)
        ssmv.ssmv_cache_reset(dims, cache.c, None, None)
        run = lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, dt=dt, Bm=B, Cm=C, A=A, D=A, L=L, y_out=y, z=gate)
        assert launches(run)[0] == (H * batch, _threads(P, N)[OTHER])
        run()
        out.append(y)
    assert torch.equal(out[0], out[1])
