"""GPU parity of the small kernels around the recurrence at the edges of their steps and tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_15237_amd as ssmv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 7, 8, 9, 16, 17, 40])
def test_first_conflict_at_every_position(k):
    """Sequence b disagrees first at position b (the last one nowhere), and again behind it."""
    batch = k + 1
    draft = np.random.default_rng(k).integers(0, 5, size=(batch, k)).astype(np.int32)
    target = draft.copy()
    for b in range(k):
        target[b, b] += 1
        target[b, b + 1::2] -= 7
    out = torch.full((batch,), -1, dtype=torch.int32, device="cuda")
    ssmv.ssmv_first_conflict(torch.from_numpy(draft).to("cuda"), torch.from_numpy(target).to("cuda"), batch, k, out)
    assert np.array_equal(out.cpu().numpy(), oracle.first_conflict(draft, target)) and out.tolist() == list(range(k + 1))


@pytest.mark.parametrize("batch,k", [(1, 64), (5, 64), (3, 65), (2, 130), (131, 33), (70, 21), (65, 63), (70000, 1), (700001, 3), (40000, 64), (33000, 40)])
def test_first_conflict_of_many_sequences(batch, k):
    """A wave's share of the lanes: sequences that fill it, leave lanes over or are longer; several shares per wave; a last one that
    is not full."""
    g = torch.Generator(device="cuda").manual_seed(batch + k)
    draft = torch.randint(0, 3, (batch, k), dtype=torch.int32, device="cuda", generator=g)
    target = draft.clone()
    at = torch.randint(0, k + 1, (batch,), device="cuda", generator=g)
    behind = torch.arange(k, device="cuda")[None] >= at[:, None]
    target[behind] = torch.randint(0, 3, (int(behind.sum()),), dtype=torch.int32, device="cuda", generator=g)
    out = torch.full((batch + 1,), -1, dtype=torch.int32, device="cuda")
    ssmv.ssmv_first_conflict(draft, target, batch, k, out)
    want = (draft == target).int().cumprod(1).sum(1).int()
    assert torch.equal(out[:batch], want) and out[batch] == -1


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("rows,groups,vecs", [(1, 1, 1), (3, 5, 7), (9, 3, 63), (5, 2, 64), (5, 2, 65), (3, 3, 80), (7, 1, 128), (2, 3, 129), (3, 1, 256),
                                              (2, 2, 257), (3, 1, 512), (2, 1, 513), (1, 2, 1024), (2050, 9, 3), (4097, 5, 80), (4099, 3, 129)])
def test_gated_rmsnorm_vector_counts(rows, groups, vecs, io):
    """Group sizes around one, two and four vectors per thread of 64, 128 and 256 threads; a last workgroup with fewer groups
    or rows than it has room for; in place as well."""
    dt, ev = (torch.bfloat16, 8) if io == "bf16" else (torch.float32, 4)
    group = vecs * ev
    ch = groups * group
    g = torch.Generator(device="cuda").manual_seed(rows * 1000 + vecs)
    y, z = (torch.randn(rows, ch, generator=g, device="cuda").to(dt) for _ in range(2))
    w = 1 + 0.1 * torch.randn(ch, generator=g, device="cuda")
    for zz in (None, z):
        v = y.double() if zz is None else y.double() * z.double() * torch.sigmoid(z.double())
        v = v.view(rows, groups, group)
        ref = (v * torch.rsqrt((v * v).mean(-1, keepdim=True) + 1e-5)).view(rows, ch) * w.double()
        out, guard = torch.zeros_like(y), y.clone()
        ssmv.ssmv_gated_rmsnorm(guard, zz, w, rows, ch, group, 1e-5, io, out)
        # one rounding to the I/O type (2^-9), or a few fp32 roundings and the hardware's exp2, rcp and rsq (an ulp each)
        tol = 2.0 ** -8 if io == "bf16" else 4e-6
        assert ((out.double() - ref).abs() <= tol * ref.abs() + 1e-30).all()
        ssmv.ssmv_gated_rmsnorm(guard, zz, w, rows, ch, group, 1e-5, io, guard)
        assert torch.equal(guard, out)


@pytest.mark.parametrize("mode,H,P,N,io,kmax", [("diag", 1, 1, 16, "bf16", 1), ("diag", 3, 1, 16, "f32", 1), ("diag", 37, 1, 32, "bf16", 4), ("scalar", 3, 5, 16, "bf16", 1),
                                                ("scalar", 3, 64, 32, "bf16", 4), ("scalar", 2, 192, 128, "bf16", 5), ("scalar", 5, 64, 64, "f32", 16)])
def test_reset_of_a_used_cache(mode, H, P, N, io, kmax):
    """Everything a cache holds is overwritten, with and without a given start; nothing is written past its buffers."""
    batch, dt = 3, torch.bfloat16 if io == "bf16" else torch.float32
    d = ssmv.make_dims(batch, H, P, N, kmax=kmax, io=io, a_mode=mode)
    g = torch.Generator(device="cuda").manual_seed(1)
    h0, conv = torch.randn(batch, H, P, N, generator=g, device="cuda"), torch.randn(batch, 3, H * P, generator=g, device="cuda").to(dt)
    A = -torch.rand(*((H, N) if mode == "diag" else (H,)), generator=g, device="cuda")
    n_ring = batch * d.ring_len * H * P
    for h, c in ((h0, conv), (None, None), (h0, None), (None, conv)):
        cache = ssmv.LayerCache.allocate(d)
        for b in cache.buffers.values():
            b.fill_(0x0101010101010101)
        ssmv.ssmv_cache_reset(d, cache.c, h, c)
        out = torch.full_like(h0, 7.0)
        ssmv.ssmv_materialize(d, cache.c, A, out)
        assert torch.equal(out, h0 if h is not None else torch.zeros_like(h0))
        ring = cache.buffers["conv_ring"].view(dt)
        want = torch.zeros(batch, d.ring_len, H * P, dtype=dt, device="cuda")
        if c is not None:
            want[:, :3] = conv
        assert torch.equal(ring[:n_ring].view_as(want), want)
        assert (cache.buffers["conv_ring"].view(torch.uint8)[n_ring * dt.itemsize:] == 1).all()
        assert (cache.buffers["state"].view(torch.uint8)[h0.numel() * 4:] == 1).all()
        i = cache.ints()
        assert [i[n].tolist() for n in ("cur_slot", "pend", "conv_head", "last_k", "pos")] == [[0] * 3, [0] * 3, [2] * 3, [0] * 3, [0] * 3]
        assert i["win_par"] == 0 and i["err_flag"] == 0


@pytest.mark.parametrize("P,N,G,io,mode,kmax", [(64, 32, 1, "bf16", "both", 8), (64, 128, 2, "bf16", "defer", 4), (192, 64, 1, "bf16", "hj_only", 8), (128, 64, 2, "bf16", "defer", 2),
                                                (20, 16, 1, "f32", "both", 16), (70, 256, 2, "f32", "hj_only", 16), (5, 128, 1, "bf16", "hj_only", 16), (64, 64, 1, "f32", "defer", 4),
                                                (128, 32, 4, "f32", "both", 5)])
def test_materialize_folds_the_pending_tokens(P, N, G, io, mode, kmax):
    """Against the vector verify kernel's replay (an explicitly chosen launch shape takes it), at every pending count that comes
    up, with the step-size transform, and with one head whose decay underflows."""
    H, batch = 4, 6
    dt = torch.bfloat16 if io == "bf16" else torch.float32
    d = ssmv.make_dims(batch, H, P, N, ngroups=G, kmax=kmax, io=io, snapshot_mode=mode)
    g = torch.Generator(device="cuda").manual_seed(2)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    A, D, w, bias, dtb = -torch.exp(rn(H)), rn(H), rn(H * P, 4).to(dt), rn(H * P).to(dt), 0.3 * rn(H)
    A[1] = -1e4
    cache = ssmv.LayerCache.allocate(d)
    ssmv.ssmv_cache_reset(d, cache.c, rn(batch, H, P, N), rn(batch, 3, H * P).to(dt))
    seen = set()
    for rnd in range(8):
        y = torch.empty(batch, kmax, H * P, dtype=dt, device="cuda")
        ssmv.ssm_block_multistep(d, cache.c, x_raw=rn(batch, kmax, H * P).to(dt), conv_wgt=w, conv_bias=bias, dt=(rn(batch, kmax, H) - 3).to(dt), dt_bias=dtb,
                                 dt_softplus=True, Bm=(rn(batch, kmax, G, N) / N ** 0.5).to(dt), Cm=rn(batch, kmax, G, N).to(dt), A=A, D=D, k=kmax, y_out=y)
        ssmv.ssm_commit_rollback(d, cache.c, torch.randint(0, kmax + 1, (batch,), generator=g, device="cuda").int())
        seen |= set(cache.ints()["pend"].tolist())
        out, ref = torch.full((batch, H, P, N), 7.0, device="cuda"), torch.full((batch, H, P, N), 9.0, device="cuda")
        ssmv.ssmv_materialize_block(d, cache.c, A, dtb, True, out)
        ssmv.ssmv_set_tuning(1, 1)
        try:
            ssmv.ssmv_materialize_block(d, cache.c, A, dtb, True, ref)
        finally:
            ssmv.ssmv_set_tuning(0, 0)
        # fp32 on both sides: a few dozen roundings of 2^-24 against the head's rms
        rms = ref.pow(2).mean((2, 3), keepdim=True).sqrt()
        assert ((out - ref).abs() / (ref.abs() + rms + 1e-30)).max() <= 4e-6
    assert len(seen) >= 3 and max(seen) >= min(kmax - 1, 3)


@pytest.mark.parametrize("io,P,N", [("f32", 20, 64), ("f32", 64, 64), ("bf16", 64, 64), ("f32", 70, 128), ("f32", 3, 256), ("bf16", 37, 256), ("bf16", 40, 128)])
@pytest.mark.parametrize("pending", [1, 3])
@pytest.mark.parametrize("A", [-3e38, -float("inf")])
def test_materialize_of_a_head_that_keeps_only_its_newest_token(A, pending, io, P, N):
    """exp(dt A) = 0: the state is dt x B^T of the last pending token, also where A log2 e is beyond fp32's range."""
    H, batch, k = 2, 2, 4
    dt = torch.bfloat16 if io == "bf16" else torch.float32
    d = ssmv.make_dims(batch, H, P, N, kmax=k, io=io, snapshot_mode="hj_only")
    g = torch.Generator(device="cuda").manual_seed(pending)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    As, D, xc, B = torch.tensor([A, A], device="cuda"), rn(H), rn(batch, k, H * P).to(dt), rn(batch, k, 1, N).to(dt)
    step = (0.1 + torch.rand(batch, k, H, generator=g, device="cuda")).to(dt)
    cache = ssmv.LayerCache.allocate(d)
    ssmv.ssmv_cache_reset(d, cache.c, rn(batch, H, P, N), None)
    ssmv.ssm_verify_multistep(d, cache.c, xc, step, B, rn(batch, k, 1, N).to(dt), As, D, k, torch.empty_like(xc))
    ssmv.ssm_commit_rollback(d, cache.c, torch.full((batch,), pending, dtype=torch.int32, device="cuda"))
    out = torch.full((batch, H, P, N), 7.0, device="cuda")
    ssmv.ssmv_materialize(d, cache.c, As, out)
    n = pending - 1
    want = (step[:, n, :, None].double() * xc[:, n].double().view(batch, H, P))[..., None] * B[:, n, 0].double()[:, None, None]
    assert ((out.double() - want).abs() <= 2.0 ** -22 * want.abs() + 1e-30).all()          # two products, an ulp each


def test_default_stream_argument_follows_torch():
    """No stream given: the current stream of the current device, whatever it is when the call is made, in every thread."""
    import threading
    from paper_2408_15237_amd.binding import _stream
    now = lambda: torch.cuda.current_stream().cuda_stream or None
    side = torch.cuda.Stream()
    assert _stream(None) == now()
    with torch.cuda.stream(side):
        assert _stream(None) == now() == side.cuda_stream
        seen = []
        th = threading.Thread(target=lambda: seen.append((_stream(None), now())))      # a thread starts on the default stream
        th.start()
        th.join()
        assert seen[0][0] == seen[0][1] != side.cuda_stream
    assert _stream(None) == now() and _stream(0) is None and _stream(side.cuda_stream) == side.cuda_stream
