"""The tile that a dense linear layer takes by its size, asked of the library's own rule (host only): the launches that
test_gpu_lin_tiles.py compares bit for bit do take different tiles, and together all of them."""
import subprocess
from pathlib import Path

import pytest

from paper_2510_05367_amd import build as lcbuild
from tests.test_gpu_lin_tiles import SPLITS

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "lc_lin_epi.h"
using namespace lc;
int main(int n, char** v) {  // rows, K, N, fp32 output, gated, ...
  for (int i = 1; i + 4 < n; i += 5) {
    Lin2Args a;
    memset(&a, 0, sizeof a);
    static float gate;
    a.rows = atoll(v[i]); a.K = atoi(v[i + 1]); a.N = atoi(v[i + 2]); a.gate = atoi(v[i + 4]) ? &gate : nullptr;
    static const char* const name[] = {"64x64", "64x128", "128x128", "256x192", "256x256", "128x160"};
    puts(name[(int)lin3_tile(a, atoi(v[i + 3]))]);
  }
}
"""


@pytest.fixture(scope="module")
def tile_of(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("tiles")
    (tmp / "ask.hip").write_text(PROGRAM)
    lib = Path(lcbuild.LIB)
    if not lib.exists():
        lcbuild.build_library()
    subprocess.run([lcbuild._hipcc(), *lcbuild.FLAGS, "-I", str(Path(lcbuild.CSRC)), str(tmp / "ask.hip"), "-o", str(tmp / "ask"), "-L", str(lib.parent),
                    "-llightcache", f"-Wl,-rpath,{lib.parent}"], check=True, capture_output=True)

    def ask(launches):
        out = subprocess.run([str(tmp / "ask"), *(str(int(v)) for l in launches for v in l)], check=True, capture_output=True, text=True, timeout=60)
        return out.stdout.split()
    return ask


def layers(rows, D):
    """rows, K, N, fp32 output, gated of a block's q,k,v, output projection and MLP"""
    return [(rows, D, 3 * D, 0, 0), (rows, D, D, 1, D % 128 == 0), (rows, D, 4 * D, 0, 0), (rows, 4 * D, D, 1, D % 128 == 0)]


def test_compared_launches_take_different_tiles(tile_of):
    seen = set()
    for B, T, D, _, groups in SPLITS:
        whole = tile_of(layers(B * T, D))
        for n in groups:
            part = tile_of(layers(n * T, D))
            assert sum(a != b for a, b in zip(whole, part)) >= 2, (B, T, D, n, whole, part)
            seen |= set(part)
        seen |= set(whole)
    assert seen == {"64x64", "64x128", "128x128", "256x192", "256x256", "128x160"}
