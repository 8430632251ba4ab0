"""The pipelined fp32 prefill kernel (csrc/prefill_f32_pipe.hip) against the oracle: every tile, heads taken whole and as parts, at the
edges of chunks and over the buffers' rotation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_15237_amd as ssmv

from _harness import TOL, launches, rel_err, to_host

pytestmark = pytest.mark.gpu


def _threads(P, N):
    """Threads of a workgroup that owns P channels: consumers, three weight waves, the decay wave, four conv waves."""
    tiles, shares = P // 32, min(max(N // 32, 1), 4 // (P // 32))
    return 64 * (tiles * shares + 8)


# (headdim, dstate, parts, batch of four heads)
CASES = [(P, N, 1, 64 if P > 32 else 3) for P in (32, 64, 128) for N in (32, 64, 128) if (P, N) != (128, 128)]
CASES += [(64, N, 2, 2) for N in (32, 64, 128)] + [(128, N, 2, 32) for N in (32, 64, 128)] + [(128, N, 4, 3) for N in (32, 64, 128)]


@pytest.mark.parametrize("block", [False, True], ids=["plain", "block"])
@pytest.mark.parametrize("P,N,parts,batch", CASES)
def test_against_the_oracle(P, N, parts, batch, block):
    """block: SiLU, gate (outputs over it), softplus, conv bias, row-major slots, lengths that differ; plain: none of it."""
    H, G = 4, 2
    g = torch.Generator(device="cuda").manual_seed(P + N + parts + block)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    Cx, seqs = H * P, [0, batch - 1]
    w, bias, D, dtb = rnd(Cx, 4) / 2, rnd(Cx) * 0.1 if block else None, rnd(H), torch.rand(H, generator=g, device="cuda") - 0.5
    A = -torch.exp(torch.rand(H, generator=g, device="cuda") * 2.7)
    act, host = "silu" if block else "none", to_host
    dims = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=4, io="f32", conv_act=act, engine="vector" if block else "auto")
    for L in (1, 31, 32, 33, 65, 161):
        h0, conv0 = rnd(batch, H, P, N) * 0.1, rnd(batch, 3, Cx)
        cache = ssmv.LayerCache.allocate(dims)
        ssmv.ssmv_cache_reset(dims, cache.c, h0, conv0)
        lens = torch.randint(0, L + 1, (batch,), generator=torch.Generator().manual_seed(L), dtype=torch.int32) if block else torch.full((batch,), L, dtype=torch.int32)
        lens[0] = L
        oras = [oracle.EagerOracle("scalar", host(A), host(D), host(w), host(bias) if block else None, host(h0[b:b + 1]), "f32", act, G,
                                   conv_init=host(conv0[b:b + 1]), dt_bias=host(dtb) if block else None, dt_softplus=block) for b in seqs]
        for _ in range(2):                                             # the second prompt continues the ring and the state of the first
            x, B, C, z = rnd(batch, L, Cx), rnd(batch, L, G, N) / N ** 0.5, rnd(batch, L, G, N) / N ** 0.5, rnd(batch, L, Cx)
            dt = rnd(batch, L, H) - 4 if block else torch.nn.functional.softplus(rnd(batch, L, H) - 4)
            y, lens_dev = z.clone() if block else torch.full_like(x, 7.0), lens.cuda() if block else None
            run = lambda: ssmv.ssm_prefill_block(dims, cache.c, x_raw=x, conv_wgt=w, conv_bias=bias, dt=dt, dt_bias=dtb if block else None, dt_softplus=block, Bm=B, Cm=C,
                                                 z=y if block else None, A=A, D=D, L=L, y_out=y, seq_len=lens_dev)
            assert launches(run)[0] == (H * batch * parts, _threads(P // parts, N)), "L = %d" % L
            run()
            h = torch.empty_like(h0)
            ssmv.ssmv_materialize_block(dims, cache.c, A, dtb if block else None, block, h)
            for ora, b in zip(oras, seqs):
                n = int(lens[b])
                if n:
                    f = lambda t: host(t[b:b + 1, :n])
                    y_ref, _, _ = ora.verify(f(x), f(dt), f(B), f(C), z=f(z) if block else None)
                    ora.commit([n])
                    assert rel_err(f(y), y_ref) <= TOL["f32"], "L = %d, sequence %d" % (L, b)
                assert torch.equal(y[b, n:], z[b, n:] if block else torch.full_like(y[b, n:], 7.0)), "L = %d: outputs behind a sequence's length" % L
                assert rel_err(host(h[b:b + 1]), ora.h) <= TOL["f32"], "L = %d, sequence %d: state" % (L, b)
        ssmv.ssmv_check(cache.c)


@pytest.mark.parametrize("P,N,H,L,parts,segments", [(128, 64, 8, 1500, 2, 16), (64, 64, 20, 1500, 1, 12), (128, 128, 4, 700, 4, 5), (32, 64, 16, 1500, 1, 16)])
def test_cut_prompts_of_parts(P, N, H, L, parts, segments):
    """Few pairs and a long prompt: cut into segments by this kernel, with the parts' states between the passes, it agrees with the same
    prompt fed in two calls, and the outputs do not depend on what was in y."""
    g = torch.Generator(device="cuda").manual_seed(P + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    dims = ssmv.make_dims(1, H, P, N, kmax=4, io="f32")
    x, B, C, w, A, D = rnd(1, L, H * P), rnd(1, L, 1, N) / N ** 0.5, rnd(1, L, 1, N) / N ** 0.5, rnd(H * P, 4) / 2, -torch.exp(torch.rand(H, generator=g, device="cuda")), rnd(H)
    dt, h0 = torch.nn.functional.softplus(rnd(1, L, H) - 4), rnd(1, H, P, N)

    def feed(cuts, fill):
        cache = ssmv.LayerCache.allocate(dims)
        ssmv.ssmv_cache_reset(dims, cache.c, h0, torch.zeros(1, 3, H * P, device="cuda"))
        ys = []
        for a, b in zip(cuts, cuts[1:]):
            y = torch.full((1, b - a, H * P), fill, device="cuda")
            tok = [t[:, a:b].contiguous() for t in (x, dt, B, C)]
            run = lambda: ssmv.ssm_prefill_chunked(dims, cache.c, tok[0], w, None, tok[1], tok[2], tok[3], A, D, b - a, y)
            if b - a == L:                                             # the segments but the last, the last one's states put together, all of them again
                launched = launches(run)
                assert len(launched) == 3 and launched[0] == (H * parts * (segments - 1), _threads(P // parts, N))
            run()
            ys.append(y)
        h = torch.empty_like(h0)
        ssmv.ssmv_materialize_block(dims, cache.c, A, None, False, h)
        return torch.cat(ys, 1), h

    y, h = feed([0, L], float("nan"))
    y1, h1 = feed([0, L], 0.0)
    assert torch.equal(y, y1) and torch.equal(h, h1)
    y2, h2 = feed([0, 37, L], 0.0)                                     # two evaluations, each within the tolerance of the exact one
    assert rel_err(host_d(y), host_d(y2)) <= 2 * TOL["f32"] and rel_err(host_d(h), host_d(h2)) <= 2 * TOL["f32"]


def host_d(t):
    return t.double().cpu().numpy().astype(np.float64)
