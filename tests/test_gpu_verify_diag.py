"""GPU parity of the quad-per-channel verify kernel of diagonal-A mode (csrc/verify_diag.hip) where its layout could go wrong:
channel counts around a wave's and a workgroup's share, odd ones (two channels per quad need an even count), draft and pending
counts around the groups of four, all snapshot modes, tokens that are not taken, and conv rings of more than 4 GiB."""
import numpy as np
import pytest
import torch

import paper_2408_15237_amd as ssmv
from workload import Workload, generate

from _harness import HipLayer, TOL, rel_err, run_parity, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("H,N", [(1, 16), (2, 16), (33, 16), (64, 16), (130, 16), (2050, 16), (17, 32), (66, 32), (15, 64), (129, 64)])
def test_channel_counts(H, N, io):
    wl = Workload("chan", "diag", batch=3, nheads=H, headdim=1, dstate=N, k=5, rounds=6, io=io, accept="uniform", seed=H)
    for fused in (False, True):
        run_parity(wl, generate(wl), fused=fused, reverify=True)


@pytest.mark.parametrize("mode,kmax", [("both", 1), ("both", 4), ("both", 5), ("both", 8), ("both", 9), ("both", 16), ("hj_only", 4), ("hj_only", 8),
                                       ("hj_only", 16), ("defer", 2), ("defer", 4), ("defer", 7), ("defer", 8)])
@pytest.mark.parametrize("accept", ["uniform", "geometric"])
def test_token_counts(mode, kmax, accept):
    wl = Workload("tok", "diag", batch=5, nheads=70, headdim=1, dstate=16, k=kmax, rounds=14, io="bf16", accept=accept, conv_act="silu",
                  seed=kmax, snapshot_mode=mode)
    run_parity(wl, generate(wl), fused=True)


@pytest.mark.parametrize("io,H", [("bf16", 66), ("bf16", 65), ("f32", 66)])
def test_tokens_not_taken_and_strong_decay(io, H):
    """Whatever stands in the tokens behind a sequence's draft count must not reach it, and A of -inf decays to nothing."""
    k, N, batch = 7, 16, 6
    wl = Workload("nan", "diag", batch=batch, nheads=H, headdim=1, dstate=N, k=k, rounds=1, io=io, accept="uniform", seed=3)
    data = generate(wl)
    lp, rd = data.layers[0], data.rounds[0]
    lp.A[::3, ::2] = -np.inf
    counts = np.array([1, 2, 4, 5, 6, 7], dtype=np.int32)
    outs = []
    for poison in (0.0, np.nan):
        hip = HipLayer(wl, lp)
        arr = [np.array(a, dtype=np.float32, copy=True) for a in (rd.x_raw, rd.dt[0], rd.B[0], rd.C[0])]
        for a in arr:
            for b in range(batch):
                a[b, counts[b]:] = poison
        x, dt, B, C = (to_dev(a, io) for a in arr)
        y = torch.empty_like(x)
        ssmv.ssm_block_multistep(hip.dims, hip.cache.c, x_raw=x, conv_wgt=hip.conv_w, conv_bias=hip.conv_b, dt=dt, Bm=B, Cm=C, A=hip.A, D=hip.D, k=k,
                                 k_seq=torch.from_numpy(counts).to("cuda"), y_out=y)
        hip.commit(torch.from_numpy(counts).to("cuda"))
        outs.append((to_host(y), to_host(hip.materialize())))
    (y0, h0), (y1, h1) = outs
    assert np.all(np.isfinite(y1)) and np.all(np.isfinite(h1))
    assert np.array_equal(y0, y1) and np.array_equal(h0, h1)
    assert np.all(y1[0, 1:] == 0)


def test_kernel_and_forced_shape_agree():
    """The same round on the quad kernel and on the LDS-staged kernel (an explicitly chosen launch shape)."""
    wl = Workload("two", "diag", batch=2, nheads=300, headdim=1, dstate=32, k=6, rounds=5, io="f32", accept="uniform", seed=8)
    data = generate(wl)
    res = []
    for tune in ((0, 0), (1, 2)):
        ssmv.ssmv_set_tuning(*tune)
        try:
            hip = HipLayer(wl, data.layers[0])
            ys = []
            for rd in data.rounds:
                y, _ = hip.conv_verify(*(to_dev(a, "f32") for a in (rd.x_raw, rd.dt[0], rd.B[0], rd.C[0])))
                ys.append(to_host(y))
                hip.commit(torch.from_numpy(rd.accepted.astype(np.int32)).to("cuda"))
            res.append((np.stack(ys), to_host(hip.materialize()), hip.cache.ints()))
        finally:
            ssmv.ssmv_set_tuning(0, 0)
    assert rel_err(res[0][0], res[1][0]) <= TOL["f32"] and rel_err(res[0][1], res[1][1]) <= TOL["f32"]
    assert res[0][2]["pend"].tolist() == res[1][2]["pend"].tolist()


@pytest.mark.parametrize("forced", [False, True])
@pytest.mark.parametrize("mode,H,P,ring_len", [("diag", 1030, 1, 1 << 20), ("diag", 64, 1, 1 << 24), ("scalar", 4, 16, 1 << 24)])
def test_ring_of_more_than_4_gib(mode, H, P, ring_len, forced):
    """The fused conv finds its history and appends its inputs where conv1d_state_update does, also in rows whose byte offset does
    not fit 32 bits or whose number does not fit the 24-bit multiplier."""
    k, N, ch = 4, 16, H * P
    d = ssmv.make_dims(1, H, P, N, kmax=k, ring_len=ring_len, io="f32", a_mode=mode)
    g = torch.Generator(device="cuda").manual_seed(ring_len)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    A, D, w, h0, x, hist = -torch.exp(rn(*((H, N) if mode == "diag" else (H,)))), rn(H), rn(ch, 4), rn(1, H, P, N), rn(1, k, ch), rn(3, ch)
    dt, B, C = 0.1 * torch.exp(rn(1, k, H)), rn(1, k, 1, N), rn(1, k, 1, N)
    ys = []
    for fused in (False, True):
        cache = ssmv.LayerCache.allocate(d)
        ssmv.ssmv_cache_reset(d, cache.c, h0, None)
        ring = cache.buffers["conv_ring"].view(torch.float32)[:ring_len * ch].view(ring_len, ch)
        ring[ring_len - 4:ring_len - 1] = hist
        cache.buffers["conv_head"].view(torch.int32)[0] = ring_len - 2
        y = torch.empty_like(x)
        if fused:
            ssmv.ssmv_set_tuning(*((1, 2) if forced else (0, 0)))
            try:
                ssmv.ssm_conv_verify_multistep(d, cache.c, x, w, None, dt, B, C, A, D, k, y)
            finally:
                ssmv.ssmv_set_tuning(0, 0)
        else:
            xc = torch.empty_like(x)
            ssmv.conv1d_state_update(d, cache.c, x, w, None, k, xc)
            ssmv.ssm_verify_multistep(d, cache.c, xc, dt, B, C, A, D, k, y)
        ys.append(to_host(y))
        assert torch.equal(ring[ring_len - 1], x[0, 0]) and torch.equal(ring[:3], x[0, 1:])
        assert torch.equal(ring[ring_len - 4:ring_len - 1], hist) and int(ring.count_nonzero()) == 7 * ch
        del cache, ring
    assert rel_err(ys[1], ys[0]) <= TOL["f32"]
