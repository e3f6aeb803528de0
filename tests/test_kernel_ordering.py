"""What the order of instructions has to guarantee, from the AMD assembly that the compiler makes of the sources (no
GPU needed).

LDS reads and stage refills in the forward product's kernels: their ring has three stages, and one barrier per step
both announces the stage that has arrived and releases the stage just read for the transfers of the step after the
next.  So a wave must have all of its LDS reads back when it arrives at a barrier: a read still on its way could meet
the refill of its stage.

Stores of 16 bytes written as assembly: the hardware wants two wait states before a vector instruction overwrites such a
store's data, and the compiler, which keeps them behind its own stores, does not look into a statement."""
import os
import re
import subprocess

import pytest

from paper_2502_05003_amd import build


def reads_outstanding_at_barriers(assembly):
    """{kernel: [LDS reads issued and not waited for, at each barrier in program order]}"""
    found, kernel, outstanding = {}, None, 0
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        label = re.match(r"(_Z\w+):", line)
        if label:
            kernel, outstanding = label.group(1), 0
            found[kernel] = []
        elif line.startswith("ds_read"):
            outstanding += 1
        elif line.startswith("s_waitcnt"):
            wait = re.search(r"lgkmcnt\((\d+)\)", line)
            if wait:
                outstanding = min(outstanding, int(wait.group(1)))
        elif line.startswith("s_barrier"):
            found[kernel].append(outstanding)
    return found


def test_the_count_on_a_sample():
    sample = """
_Zk:
	ds_read_b128 v[0:3], v9
	ds_read_b128 v[4:7], v9 offset:64
	s_waitcnt vmcnt(4) lgkmcnt(1)
	s_barrier                       ; one read may be on its way
	s_waitcnt lgkmcnt(0)
	s_barrier
"""
    assert reads_outstanding_at_barriers(sample) == {"_Zk": [1, 0]}


@pytest.mark.parametrize("source,kernels", [("fp4_gemm.hip", 2), ("lowbit_gemm.hip", 6)])
def test_no_read_is_outstanding_at_a_barrier(source, kernels, tmp_path):
    out = str(tmp_path / "kernels.s")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get(source, []), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    found = {k: v for k, v in reads_outstanding_at_barriers(open(out).read()).items()
             if re.search(r"gemm_(tile|wide|small)_kernel", k)}
    assert len(found) == kernels and all(len(v) >= 3 for v in found.values())
    assert {k: v for k, v in found.items() if any(v)} == {}


SIXTEEN_BYTE_STORE = r"""
#include "quest_device.h"
__global__ void overwrites_the_data(uint32_t *p)
{
    quest::quest_v4u v = {p[0], p[1], p[2], p[3]};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        quest::store_16_counted(p + 1024 * i, 16 * threadIdx.x, v);
        asm volatile("v_add_u32 %0, 1, %0" : "+v"(v));   // the very next instruction
    }
}
"""


def wait_states_behind_stores(assembly):
    """For each 16-byte store: instructions, s_nop by its count, up to the next vector instruction."""
    found, behind = [], None
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        if behind is not None:
            nop = re.match(r"s_nop (\d+)", line)
            if line.startswith("v_"):
                found.append(behind)
                behind = None
            else:
                behind += 1 + (int(nop.group(1)) if nop else 0)
        if line.startswith("global_store_dwordx4"):
            behind = 0
    return found


def test_sixteen_byte_stores_keep_their_data(tmp_path):
    source, out = tmp_path / "store.hip", tmp_path / "store.s"
    source.write_text(SIXTEEN_BYTE_STORE)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.HIPCC_FLAGS, "-I" + build.CSRC, "--cuda-device-only", "-S", str(source), "-o", str(out)],
                   check=True, capture_output=True)
    states = wait_states_behind_stores(out.read_text())
    assert len(states) == 8 and min(states) >= 2, states
