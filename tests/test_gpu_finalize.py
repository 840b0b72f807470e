"""Folding GroupNorm partial sums: groups with an odd number of channels (one channel a load), the concatenation's groups across
its two sources, and frames with so many splits that the launch takes 1024 threads, through a residual block and the up
convolution against the oracle."""
import re
from pathlib import Path

import numpy as np
import pytest

from oracle import lightcache_oracle as lo
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import build as lcbuild
from paper_2510_05367_amd import synth
from tests.gpu_util import check, dev, dev32, empty32, host, make_stage, planar_to_rows, rows_to_planar

pytestmark = pytest.mark.gpu


def threads(C, groups, rows):
    """of the launch that folds a group's statistics (single operators take them in splits of 64 rows)"""
    line = int(re.search(r"const int nt = cells > (\d+) \? 1024 : 256;", (Path(lcbuild.CSRC) / "lc_norm.hip").read_text()).group(1))
    cg, splits = C // groups, -(-rows // 64)
    return 1024 if cg * splits // (2 if cg % 2 == 0 else 1) > line else 256


# 320 / 64 = 5 channels a group, 448 / 64 = 7 over both sources (one group has channels of both); 10 and 12 with two channels a
# load; frames of one split, of 96 x 128 pixels = 192 splits (960 to 1344 loads of a group, 256 threads) and of 160 x 128 = 320
# splits (1600 to 2240 loads, 1024 threads)
@pytest.mark.parametrize("C,Cd,heads,hd,groups,H,W,nt", [(320, 128, 5, 64, 64, 6, 10, 256), (320, 128, 5, 64, 64, 96, 128, 256), (320, 64, 5, 64, 32, 96, 128, 256),
                                                         (320, 128, 5, 64, 64, 160, 128, 1024), (320, 64, 5, 64, 32, 160, 128, 1024)])
def test_odd_groups_and_many_splits(C, Cd, heads, hd, groups, H, W, nt):
    assert threads(C, groups, H * W) == threads(C + Cd, groups, H * W) == nt
    cfg = synth.StageConfig("fin", B=1, F=1, H=H, W=W, C_lat=4, C=C, C_deep=Cd, groups=groups, n_res=1, heads=heads, head_dim=hd, dtype="bf16")
    print(f"[case] C {C} C_deep {Cd} {H} x {W}", flush=True)
    stage, w = make_stage(cfg, seed=3)
    w = {k: v.astype(np.float64) for k, v in w.items()}
    try:
        x = synth.make_activation((1, C, H, W), 1, "bf16", 1.5) + np.float32(0.5)
        d = synth.round_to_bf16(synth.make_activation((1, Cd, H // 2, W // 2), 2, "bf16", 0.7))
        xd, dd = dev32(stage, planar_to_rows(x)), dev(stage, planar_to_rows(d))
        y, u = empty32(stage, *xd.shape), empty32(stage, H * W, C)
        lcb.lc_op_res_block(stage.ctx, lcb.LC_L_RES0, xd.data_ptr(), y.data_ptr(), 1)
        lcb.lc_op_up_conv(stage.ctx, xd.data_ptr(), dd.data_ptr(), u.data_ptr(), 1)
        stage.sync()
        x64 = x.astype(np.float64)
        ref = x64 + lo.conv3x3(lo.silu(lo.group_norm(x64, w["res0.gn_g"], w["res0.gn_b"], groups, cfg.gn_eps)), w["res0.w"], w["res0.b"])
        check("res_block", rows_to_planar(host(y), 1, C, H, W), ref, "bf16")
        cat = np.concatenate([x64, lo.up2(d.astype(np.float64))], axis=1)
        ref = lo.conv3x3(lo.silu(lo.group_norm(cat, w["up.gn_g"], w["up.gn_b"], groups, cfg.gn_eps)), w["up.w"], w["up.b"])
        check("up_conv", rows_to_planar(host(u), 1, C, H, W), ref, "bf16")
    finally:
        stage.close()
