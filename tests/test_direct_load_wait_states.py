"""The loads that go straight into LDS (csrc/prefill_bf16_ops.h) are inline assembly, inside which the compiler resolves no hazards.  Their
base address is a scalar; on gfx9 a vector memory access may read a scalar that a vector instruction wrote (v_readfirstlane, or
v_readlane of a spilled one) only five wait states later, one that a scalar instruction wrote at once.  A probe in which such an instruction comes right ahead of the load is
compiled for the device (no GPU needed) and the wait states in between are counted."""
import re
import shutil
import subprocess

import pytest

from paper_2408_15237_amd import build

PROBE = """
#include "prefill_bf16_ops.h"
using namespace ssmv;
extern "C" __global__ void probe(const char *const *bases, float *out)
{
    __shared__ float4 lds[64];
    const size_t a = (size_t)bases[threadIdx.x];
    const size_t base = ((size_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)a);
    %s((const void *)base, threadIdx.x * 16u, (const char *)lds);
    wait_direct_loads();
    out[threadIdx.x] = lds[threadIdx.x].x;
}
"""


def _scalars(operand):
    m = re.match(r"s(?:(\d+)|\[(\d+):(\d+)\])$", operand)
    return range(0) if not m else range(int(m[1]), int(m[1]) + 1) if m[1] else range(int(m[2]), int(m[3]) + 1)


@pytest.mark.parametrize("load", ["load_to_lds16", "load_to_lds2"])
def test_five_wait_states_between_a_vector_written_base_and_the_load(load, tmp_path):
    hipcc = build._hipcc()
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE % load)
    subprocess.run([hipcc] + build.FLAGS + ["--offload-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    now, written, seen = 0, {}, []                # wait states so far; by scalar that a vector instruction wrote: those since then
    for line in asm.read_text().splitlines():
        m = re.match(r"\s+([a-z]\w+)\s*(.*)", line.split(";")[0])
        if not m:
            continue
        op, args = m[1], [a.split()[0] for a in m[2].split(",") if a.split()]
        if op.startswith("global_load_lds"):
            seen.append(min((now - written[r] for a in args for r in _scalars(a) if r in written), default=5))
        now += int(args[0], 0) + 1 if op == "s_nop" else 1
        if op.startswith("v_") and args:
            written.update((r, now) for r in _scalars(args[0]))
        elif op.startswith("s_") and args:        # waits for the vector instruction itself; what it writes may be read at any time
            for r in _scalars(args[0]):
                written.pop(r, None)
    assert any(written), "the probe's base did not come from a vector instruction"
    assert len(seen) == 1 and seen[0] >= 5, "wait states: %s" % seen
