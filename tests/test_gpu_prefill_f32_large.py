"""fp32 prefill launches of every size: which of the two kernels a call runs, whole, in parts or cut (csrc/prefill.hip: plan_f32)."""
import pytest
import torch

import paper_2408_15237_amd as ssmv

from _harness import launches

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
