"""Rows and pixels beyond the end are left to the range check of buffer loads and stores. For raw buffers it compares the
vector offset (with the immediate one) with the descriptor's size less the scalar offset, so a scalar offset beyond the size
leaves nothing defined to compare with. This test compiles the kernels whose epilogues rely on the check to gfx950 assembly:
none of their accesses (but the loads straight to LDS, whose scalar offset stays inside a row) has a scalar offset."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild

CSRC = Path(lcbuild.__file__).parent / "csrc"


@pytest.mark.parametrize("src", ["lc_lin2", "lc_lin3", "lc_conv", "lc_convd"])
def test_no_scalar_offset_where_the_range_check_decides(src, tmp_path):
    out = tmp_path / f"{src}.s"
    subprocess.run([lcbuild._hipcc(), *lcbuild.FLAGS, "-S", "--cuda-device-only", str(CSRC / f"{src}.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    accesses = [l.split(";")[0].strip() for l in out.read_text().splitlines() if re.match(r"\s+buffer_(load|store)", l)]
    accesses = [l for l in accesses if not l.endswith("lds")]
    assert accesses
    for l in accesses:
        assert re.search(r", s\[\d+:\d+\], 0 offen( offset:\d+)?$", l), l
