"""Which 3x3 convolutions of a bf16 stage run as an activation pass and the kernel over activated rows: asked of the library's own
dispatch with launches of no frames, which start nothing on a device. Rows that are only rounded (no GroupNorm in front of the
convolution) take it only where the caller says that scale and shift are those of the identity, since the pass then ignores
them; anything else goes to the kernel that applies them."""
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "lc_internal.h"
using namespace lc;
int main() {
  static char room[64];
  for (int src = 1; src <= 3; ++src)
    for (int unit = 0; unit < 2; ++unit)
      for (int scratch = 0; scratch < 2; ++scratch) {
        FusedDesc d;
        memset(&d, 0, sizeof d);
        d.dt = kBF16; d.y_f32 = 1; d.taps = 9; d.src = src; d.Cin = 128; d.Cs = 64; d.Cout = 64; d.Cout_store = 64; d.H = 8; d.W = 16;
        d.w = d.x = d.x2 = room; d.y = room; d.scale = d.shift = (const float*)room; d.unit_scale = unit;
        if (scratch) { d.xact = room; d.xact_bytes = sizeof room; }
        printf("%d %d %d %d\n", src, unit, scratch, launch_conv_act_dma(nullptr, d) == hipSuccess);
      }
}
"""


@pytest.fixture(scope="module")
def taken(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("dispatch")
    (tmp / "ask.hip").write_text(PROGRAM)
    lib = Path(lcbuild.LIB)
    if not lib.exists():
        lcbuild.build_library()
    subprocess.run([lcbuild._hipcc(), *lcbuild.FLAGS, "-I", str(Path(lcbuild.CSRC)), str(tmp / "ask.hip"), "-o", str(tmp / "ask"), "-L", str(lib.parent),
                    "-llightcache", f"-Wl,-rpath,{lib.parent}"], check=True, capture_output=True)
    out = subprocess.run([str(tmp / "ask")], check=True, capture_output=True, text=True, timeout=60).stdout
    return {tuple(map(int, l.split()[:3])): l.split()[3] == "1" for l in out.splitlines()}


def test_activation_pass_only_where_it_computes_the_same(taken):
    assert len(taken) == 12
    for (src, unit, scratch), yes in taken.items():
        assert yes == bool(scratch and (src != 1 or unit)), (src, unit, scratch)
