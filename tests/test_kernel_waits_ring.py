"""The bf16 spatial attention kernel hands LDS from one wavefront to another at barriers of its own: those inside its key
loop wait for the loads to LDS only (vmcnt), so what a wavefront wrote to LDS itself before the loop - the ones and zeros
behind V^T, whose readers are the other wavefronts - must be ordered by the first barrier, which has to wait for LDS too
(lgkmcnt(0)) right where it stands, not where the compiler happens to want some result. Checked in the compiled gfx950
assembly of every instantiation: between the last write to LDS before the first barrier and that barrier there is a wait
for all of LDS, and the barrier's own wait covers both counters."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild

CSRC = Path(lcbuild.__file__).parent / "csrc"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "lc_attn.s"
    cmd = [lcbuild._hipcc(), *lcbuild.FLAGS, "-S", "--cuda-device-only", str(CSRC / "lc_attn.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    asm = out.read_text()
    found = {}
    for name in re.findall(r"^(_ZN2lc24spatial_attn_ring_kernel[^:\n]*):", asm, flags=re.M):
        start = asm.index("\n" + name + ":")
        found[name] = asm[start:asm.index("s_endpgm", start)]
    return found


def test_first_barrier_orders_the_prologues_lds_writes(kernels):
    assert len(kernels) >= 10
    for name, body in kernels.items():
        lines = [l.split(";")[0].strip() for l in body.splitlines()]
        first = next(i for i, l in enumerate(lines) if l == "s_barrier")
        waits = []
        for l in reversed(lines[:first]):
            if l.startswith("s_waitcnt"):
                waits.append(l)
            elif l:
                break
        joined = " ".join(waits)
        assert "vmcnt(0)" in joined and "lgkmcnt(0)" in joined, (name, waits)
        writes = [i for i, l in enumerate(lines[:first]) if l.startswith("ds_write")]
        assert writes, name  # the flag at least


def test_key_loops_barriers_wait_for_the_loads_and_nothing_spills(kernels):
    """Behind the barrier of a stage every load to LDS that any wavefront issued has landed; and the two forms of the key loop
    fit the registers of two wavefronts per SIMD (a spilled loop is slow and says nothing)."""
    for name, body in kernels.items():
        assert "scratch_" not in body, f"{name}: register spills"
        assert max(int(r) for r in re.findall(r"\bv(\d+)\b", body)) < 256
        lines = [l.split(";")[0].strip() for l in body.splitlines()]
        lines = [l for l in lines if l]
        loads = [i for i, l in enumerate(lines) if l.startswith("buffer_load_dwordx4") and l.endswith("lds")]
        assert loads, name
        # in front of a barrier: a wait for every load or (__syncthreads between writes and reads of LDS) for LDS, with no
        # load to LDS and no write to it between the two; and in the stages, whose barriers follow loads, the former
        full = 0
        for i, l in enumerate(lines):
            if l == "s_barrier":
                for b in reversed(lines[:i]):
                    assert not (b.startswith("ds_write") or b in ("s_barrier",) or b.endswith("lds")), (name, lines[max(i - 8, 0):i + 1])
                    if b.startswith("s_waitcnt") and ("vmcnt(0)" in b or "lgkmcnt(0)" in b):
                        full += "vmcnt(0)" in b
                        break
                    if b.endswith(":"):
                        break
        assert full >= 4, (name, full)  # first barrier of a sweep, plain loop, safe loop, the sweep for the maxima
