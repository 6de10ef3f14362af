"""Register operands of the TIES fold's inline assembly (ties_fold2): whatever
the values it is called with, no instruction may read an input (delta,
threshold, count increment) from a register that the block has written.  Runs
on the CPU: hipcc cross-compiles a kernel whose state starts with the inputs'
own values, and the test replays the emitted block's register writes and reads."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2605_29489_amd import build

PROBE = """
#include "device_common.h"
namespace mp {
__global__ void fold_probe(const float* a, float* o, uint32_t* c)
{
    const int t = threadIdx.x;
    const float d0 = a[t], d1 = a[t + 64], tau = a[0];
    float ps0 = d0, ns0 = d1, ps1 = tau, ns1 = 0.0f;
    uint32_t c0 = 0x10000u, c1 = 0u;
    ties_fold2(d0, d1, tau, 0x10000u, ps0, ns0, c0, ps1, ns1, c1);
    o[t] = ps0; o[t + 64] = ns0; o[t + 128] = ps1; o[t + 192] = ns1;
    c[t] = c0; c[t + 64] = c1;
}
}  // namespace mp
"""


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="no hipcc")
def test_fold_reads_no_register_it_has_written(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run([build.HIPCC, *build.CFLAGS, "--cuda-device-only", "-S", "-I", build.CSRC, str(src), "-o", str(out)],
                   check=True, capture_output=True)
    blocks = re.findall(r";;#ASMSTART(.*?);;#ASMEND", out.read_text(), flags=re.S)
    assert len(blocks) == 1
    ops = [m.groups() for m in re.finditer(r"^\s*(v_\w+) ([^,]+), ([^,]+), (\S+)\s*$", blocks[0], flags=re.M)]
    compares = [o for o in ops if o[0].startswith("v_cmpx_le_f32")]
    adds = [o for o in ops if o[0] == "v_add_f32_e32"]
    counts = [o for o in ops if o[0] == "v_add_u32_e32"]
    assert (len(compares), len(adds), len(counts)) == (4, 4, 4)
    state = {o[1] for o in adds + counts}
    assert len(state) == 6  # two sums and a count per element
    inputs = {o[2] for o in compares} | {o[3].lstrip("-") for o in compares} | {o[3] for o in adds}
    inputs |= {o[2] for o in counts if not o[2].isdigit()}
    assert not state & inputs, f"the block writes inputs: {sorted(state & inputs)}"
