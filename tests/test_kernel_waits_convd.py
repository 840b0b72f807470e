"""The convolution over activated rows (lc_convd.hip) brings weights and halo lines to LDS by buffer loads and ends every
sub-step with a wait that leaves a counted number of them in flight: the weights of sub-step t + 2 must have landed, so it may
leave at most the requests issued behind theirs. This test compiles the kernel to gfx950 assembly and checks every such wait
against the requests the compiler emitted: those that every wavefront issues count, those under a condition (the left-over
weight fragments of an odd width in every other sub-step, the fifth instruction of a pair of halo lines) only as far as every
wavefront issues one in any two sub-steps. Nothing else may touch memory in the loop, nothing spills, and two workgroups fit
a compute unit."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild

CSRC = Path(lcbuild.__file__).parent / "csrc"


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "lc_convd.s"
    subprocess.run([lcbuild._hipcc(), *lcbuild.FLAGS, "-S", "--cuda-device-only", str(CSRC / "lc_convd.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    return out.read_text()


def kernels(asm):
    names = re.findall(r"^(_ZN2lc15conv_dma_kernelILi(\d)E[^:\n]*):", asm, flags=re.M)
    assert sorted(int(w) for _, w in names) == [2, 2, 3, 3, 4, 4, 5, 5]
    for name, w in names:
        start = asm.index("\n" + name + ":")
        yield name, int(w), asm[start:asm.index(".Lfunc_end", start)]


def ring_of(w):
    """weight sub-steps in LDS for a width of w channel tiles"""
    m = re.search(r"cd_ring\(\) \{ return CO_T == 2 \? (\d+) : CO_T == 3 \? (\d+) : (\d+); \}", (CSRC / "lc_convd.hip").read_text())
    return int(m.group({2: 1, 3: 2}.get(w, 3)))


def halo_pairs(t, more):
    return 1 if t == 0 or (more and t in (2, 4, 6, 12)) else 0


def test_waits_match_the_requests(asm):
    for name, w, body in kernels(asm):
        assert "scratch_" not in body, name
        ring = ring_of(w)
        steps = [p for p in body.split("s_barrier") if p.count("v_mfma") == 2 * w]
        assert len(steps) == 36, name  # 18 sub-steps of the loop over slabs and of the last slab

        def requested(t, more):
            return more or t + ring < 18  # whether sub-step t requests weights

        def at_least(n):
            return n // 2 * w + n % 2 * (w // 2)  # weight requests of every wavefront in n sub-steps in a row

        for i, p in enumerate(steps):
            t, more = i % 18, i < 18
            lds = len(re.findall(r"buffer_load_dwordx4 .* lds", p))
            # (w + 1) / 2 weight requests, and two instructions for a pair of halo lines: one by every wavefront, one by one of them
            assert lds == requested(t, more) * ((w + 1) // 2) + 2 * halo_pairs(t, more), (name, t, more)
            if i + 1 < len(steps):
                assert len(re.findall(r"\b(?:global|buffer|flat)_(?:load|store|atomic)", p)) == lds, (name, t)
            reads = p.count("ds_read_b128")
            if not more and t == 17:  # nothing follows the last sub-step
                assert reads == 0, name
                continue
            assert reads == w + 2, (name, t)
            last = [l for l in p.rstrip().splitlines() if l.strip() and not l.strip().startswith(";")][-1]
            m = re.fullmatch(r"\s*s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)\s*", last)
            assert m, (name, t, last)
            wait = int(m.group(1))
            # the weights of t + 2 were requested in sub-step t + 2 - ring, behind the halo lines of that sub-step; younger are the
            # requests of the sub-steps since (those of the slab before request no halo lines that late)
            since = [q for q in range(t + 3 - ring, t + 1)]
            younger = at_least(sum(requested(q, more or q < 0) for q in since)) + sum(halo_pairs(q, more) for q in since if q >= 0)
            assert wait <= younger, (name, t, more, wait, younger)
            # halo lines requested in sub-step 0 (12) are read during sub-step 5 (17): they have landed at the end of 4 (16)
            if t == 4 or (t == 16 and more):
                since = range(t - 4, t + 1)
                younger = at_least(sum(requested(q, more) for q in since)) + sum(halo_pairs(q, more) for q in since if q > t - 4)
                assert wait <= younger, (name, t, more, wait, younger)
            # and no stricter than that by more than the one pair of lines
            assert wait >= min(younger, at_least(ring - 2)) - 1 or not more, (name, t, wait)


def test_two_workgroups_per_compute_unit(asm):
    meta = re.findall(r"\.amdhsa_kernel (\S*conv_dma_kernel\S*)(.*?)\.end_amdhsa_kernel", asm, flags=re.S)
    assert len(meta) == 8
    for name, m in meta:
        assert int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", m).group(1)) <= 256, name
        assert int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", m).group(1)) == 0, name
    src = (CSRC / "lc_convd.hip").read_text()
    lines = int(re.search(r"constexpr int kdLines = (\d+);", src).group(1))
    for w in (2, 3, 4, 5):
        assert ring_of(w) * 2 * w * 1024 + lines * 20 * 128 <= 80 * 1024
