"""The size-chosen tiles of the dense-row linear layers (lc_lin3.hip) keep a ring of S stages filled by loads straight to
LDS. One barrier per step: its wait leaves the loads of the S - 2 stages behind the next one in flight (S - 1 before the
first step; none where K ends) and waits for every LDS read, since the stage it frees is loaded again behind it. This test
compiles the file to gfx950 assembly and checks, for every instantiation: every barrier has such a wait right in front of it,
each of the three counts occurs, the loads come in whole stages, nothing spills, and the registers leave room for the
workgroups that the launch bounds promise."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild

CSRC = Path(lcbuild.__file__).parent / "csrc"


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "lc_lin3.s"
    cmd = [lcbuild._hipcc(), *lcbuild.FLAGS, "-S", "--cuda-device-only", str(CSRC / "lc_lin3.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def test_ring_waits_match_the_stages(asm):
    names = re.findall(r"^(_ZN2lc11lin3_kernelI(?:f|DF16b)Li(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E[^:\n]*):", asm, flags=re.M)
    assert len(names) == 8
    for name, *nums in names:
        wm, wn, mt, nt, stages = map(int, nums)
        per = (32 * wm * mt + 32 * wn * nt) // 8 // (wm * wn)  # loads per wavefront and stage
        start = asm.index("\n" + name + ":")
        body = asm[start:asm.index(".Lfunc_end", start)]
        assert "scratch_" not in body, f"{name}: register spills"
        lines = [l.split(";")[0].strip() for l in body.splitlines()]
        lines = [l for l in lines if l]
        counts = set()
        for i, l in enumerate(lines):
            if l == "s_barrier":
                m = re.fullmatch(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)", lines[i - 1])
                assert m, (name, lines[i - 1])
                counts.add(int(m.group(1)))
        assert counts == {0, (stages - 1) * per, (stages - 2) * per}, (name, counts, per)
        loads = sum(l.startswith("buffer_load_dwordx4") and l.endswith("lds") for l in lines)
        assert loads == (stages + 1) * per, (name, loads, per)  # the prologue's stages and the loop's
    regs = re.findall(r"\.name:\s+(_ZN2lc11lin3_kernel\S*)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", asm)
    assert len(regs) == 8
    for name, n in regs:
        assert int(n) <= 256, name
