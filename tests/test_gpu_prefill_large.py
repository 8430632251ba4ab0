"""bf16 prefill launches of more (sequence, head) pairs than the pipelined kernel (csrc/prefill_pipe.hip) takes: which kernel a call runs."""
import pytest
import torch

import paper_2408_15237_amd as ssmv

from _harness import launches

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
