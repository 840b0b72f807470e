"""The convolution over activated rows (lc_convd.hip) at every width of its workgroups (2, 3, 4 and 5 tiles of 32 channels,
chosen by the launch's size) and at the edges of its tiles: it adds the same products in the same order as the general
kernel, which activates in its loader, so residual convolution, up convolution (two sources, one of half the resolution) and
a whole normal and cache step, whose GroupNorms read the partial sums the convolutions write, agree bit for bit."""
import pytest
import torch

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import dev, dev32, empty32, make_stage, planar_to_rows

pytestmark = pytest.mark.gpu


# C, C_deep, heads, frames, H, W: one ragged tile; narrow launches of each width; 5 x 8 tiles a frame (38 rows: a ragged last
# one; 126 columns: a ragged last tile) in as many frames as make the rule take 5, 4 and 3 channel tiles
@pytest.mark.parametrize("C,Cd,heads,F,H,W", [(64, 64, 1, 1, 6, 10), (320, 640, 5, 2, 18, 34), (192, 64, 3, 1, 8, 16), (320, 128, 5, 3, 38, 126),
                                              (128, 64, 2, 7, 38, 128), (192, 128, 3, 5, 38, 126)])
def test_rows_kernel_equals_general_bitwise(C, Cd, heads, F, H, W):
    cfg = synth.StageConfig("rows", B=1, F=F, H=H, W=W, C_lat=4, C=C, C_deep=Cd, groups=32, n_res=1, heads=heads, head_dim=C // heads,
                            dtype="bf16")
    print(f"[case] C {C} C_deep {Cd} frames {F} of {H} x {W}", flush=True)
    stage, _ = make_stage(cfg, seed=5)
    try:
        x = synth.make_activation((F, C, H, W), 1, "bf16", 1.5)
        d = synth.round_to_bf16(synth.make_activation((F, Cd, H // 2, W // 2), 2, "bf16", 0.7))
        xd, dd = dev32(stage, planar_to_rows(x)), dev(stage, planar_to_rows(d))
        lat = dev(stage, synth.make_latents(cfg, 3))
        outs = []
        for general in (1, 0):
            lcb.lc_set_conv_general(stage.ctx, general)
            y, u = empty32(stage, *xd.shape), empty32(stage, F * H * W, C)
            full, cached = stage.empty(*lat.shape), stage.empty(*lat.shape)
            lcb.lc_op_res_block(stage.ctx, lcb.LC_L_RES0, xd.data_ptr(), y.data_ptr(), F)
            lcb.lc_op_up_conv(stage.ctx, xd.data_ptr(), dd.data_ptr(), u.data_ptr(), F)
            stage.full_step(lat, full, 0)
            stage.cached_step(lat, cached, 0)
            stage.sync()
            outs.append((y, u, full, cached))
        for name, a, b in zip(("res_block", "up_conv", "normal step", "cache step"), *outs):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b), name
    finally:
        stage.close()
