"""Registers of forward kernels, as the compiler reports them for gfx950: what
a launch bound or an address held per lane costs shows here before it shows in
a time."""
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from paper_2011_13579_amd import build  # noqa: E402

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")


def _resources(tmp_path, text):
    """{template arguments: (spilled registers, wavefronts per SIMD)}"""
    src = tmp_path / "k.hip"
    src.write_text(text)
    r = subprocess.run(["hipcc"] + build.FLAGS + ["-I", build.CSRC, "-I", os.path.join(ROOT, "include"), "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c", str(src), "-o",
                        str(tmp_path / "k.o")], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    out, name = {}, None
    for ln in r.stderr.splitlines():
        if (m := re.search(r"Function Name: \S*?k_fwd_\w+?I((?:Li\d+E)+)E", ln)):
            name = tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(1)))
        elif (m := re.search(r"Occupancy.*?: (\d+)", ln)) and name:
            out[name] = (0, int(m.group(1)))
        elif (m := re.search(r"VGPRs Spill: (\d+)", ln)) and name:
            out[name] = (int(m.group(1)), out[name][1])
    return out


ROT = """#include "mivit_fwd_rot.h"
namespace mivit {
template __global__ void k_fwd_rot<%d, %d, %d, 2>(const DevCode*, const Item*, const int2*, int,
    const void*, uint64_t*, void*, int32_t*, int32_t*, int32_t*);
}
"""


@pytest.mark.parametrize("km1,dt,beta", [(5, 2, 4), (5, 0, 4), (6, 2, 4), (6, 0, 2)])
def test_rotating_kernel_keeps_its_registers(tmp_path, km1, dt, beta):
    """A period holds 32 branch metrics and the soft values of a trip: a few
    registers may go to memory around the periods, not those of a period."""
    (spill, waves), = _resources(tmp_path, ROT % (km1, dt, beta)).values()
    assert spill <= 16 and waves >= 4


def test_rate_quarter_k9_fills_the_simds(tmp_path):
    """Plans cut int8 K = 9 batches into four wavefronts per SIMD."""
    res = _resources(tmp_path, '#include "mivit_fwd_wide.hip"\n')
    assert res[(8, 4)] == (0, 4)
