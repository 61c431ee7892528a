"""Direct global->LDS loads: the chip needs a wait state between a scalar write
of M0 and an LDS load that uses it.  The loads are inline asm, so the compiler
does not put it in; this reads the gfx950 assembly of every helper."""
import glob
import os
import re
import subprocess

import pytest

from paper_2606_31808_amd import build

PROBE = """
#include "lds_dma.h"
using namespace lmop;
extern "C" __global__ void probe(const char* a, unsigned off, unsigned lds) {
  extern __shared__ char smem[];
  g2l16(a + off * threadIdx.x, smem);
  g2l16_m0(a, off * threadIdx.x, lds);
  g2l16_m0_lanes<64>(a, off * threadIdx.x, lds);
  g2l16_m0_lanes<32>(a, off * threadIdx.x, lds);
}
"""


def _m0_hazards(asm):
    """(LDS loads, those whose instruction before writes M0)"""
    loads, bad, last = 0, [], ""
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        if line.startswith("global_load_lds"):
            loads += 1
            if re.match(r"s_\w+ m0,", last):
                bad.append((last, line))
        last = line
    return loads, bad


def test_scanner_sees_the_hazard():
    load = "global_load_lds_dwordx4 v0, s[0:1]"
    assert _m0_hazards(f"s_mov_b32 m0, s2\n{load}")[1]
    assert not _m0_hazards(f"s_mov_b32 m0, s2\ns_nop 0\n{load}")[1]


def test_wait_state_after_m0(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-x", "hip", "--offload-device-only", "-S", str(src),
                    "-o", str(out)], check=True, capture_output=True)
    loads, bad = _m0_hazards(out.read_text())
    assert loads == 4
    assert not bad, bad


def test_lds_loads_only_in_the_helpers():
    for f in glob.glob(os.path.join(build.CSRC, "*")):
        if os.path.basename(f) != "lds_dma.h":
            with open(f) as src:
                assert "global_load_lds_dwordx4 %" not in src.read(), f
