"""The 3x3 convolution with specialised wavefronts (lc_convws.hip) against the general kernel and the one over activated rows,
bit for bit. It runs where a launch cannot have activated rows: on the blocks of a spatial chunk, and in single-operator calls
on more frames than the chunk scratch has room for, which is how frames of ragged tiles reach it."""
import pytest
import torch

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import dev, dev32, empty32, make_stage, planar_to_rows

pytestmark = pytest.mark.gpu


def tensors(stage, cfg):
    x = synth.make_activation((cfg.N, cfg.C, cfg.H, cfg.W), 1, "bf16", 1.5)
    d = synth.round_to_bf16(synth.make_activation((cfg.N, cfg.C_deep, cfg.H // 2, cfg.W // 2), 2, "bf16", 0.7))
    return dev32(stage, planar_to_rows(x)), dev(stage, planar_to_rows(d))


def convolutions(stage, cfg, xd, dd, general):
    lcb.lc_set_conv_general(stage.ctx, general)
    y, u = empty32(stage, *xd.shape), empty32(stage, *xd.shape)
    lcb.lc_op_res_block(stage.ctx, lcb.LC_L_RES0, xd.data_ptr(), y.data_ptr(), cfg.N)
    lcb.lc_op_up_conv(stage.ctx, xd.data_ptr(), dd.data_ptr(), u.data_ptr(), cfg.N)
    stage.sync()
    lcb.lc_set_conv_general(stage.ctx, 0)
    return y, u


# C, C_deep, heads, F, H, W: a tile's remainder in both directions, a frame smaller than a tile, two blocks of 160 channels a tile
# and four, whole tiles
@pytest.mark.parametrize("C,Cd,heads,F,H,W", [(320, 640, 5, 6, 18, 34), (320, 64, 8, 7, 6, 10), (640, 128, 10, 6, 14, 30), (320, 128, 8, 6, 16, 32)])
def test_whole_frames_beyond_the_scratch(C, Cd, heads, F, H, W):
    cfg = synth.StageConfig("ws", B=1, F=F, H=H, W=W, C_lat=4, C=C, C_deep=Cd, groups=32, n_res=1, heads=heads, head_dim=C // heads, dtype="bf16")
    print(f"[case] C {C} C_deep {Cd} frames {F} of {H} x {W}", flush=True)
    # the scratch of a chunk of one frame: 10 bytes a pixel and channel and 2 for each of the V^T rows' columns, which come in
    # 64s. What the rows would lie behind, 4 bytes a pixel and channel of all frames, is more
    T = H * W
    assert 4 * F * T > 10 * T + 2 * ((T + 63) // 64 * 64) + 8
    stage, _ = make_stage(cfg, seed=5, frame_chunk=1)
    try:
        xd, dd = tensors(stage, cfg)
        special, general = (convolutions(stage, cfg, xd, dd, g) for g in (0, 1))
        stage.set_chunk(0, 0)
        rows = convolutions(stage, cfg, xd, dd, 0)
        for name, a, b, c in zip(("residual", "up"), special, general, rows):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b) and torch.equal(a, c), name
    finally:
        stage.close()


@pytest.mark.parametrize("eta,omega", [(1, 2), (3, 1), (3, 2)])
def test_spatial_blocks(eta, omega):
    cfg = synth.StageConfig("ws", B=1, F=3, H=24, W=64, C_lat=4, C=320, C_deep=128, groups=32, n_res=1, heads=8, head_dim=40, dtype="bf16")
    stage, _ = make_stage(cfg, seed=5)
    try:
        xd, dd = tensors(stage, cfg)
        rows = convolutions(stage, cfg, xd, dd, 0)
        stage.set_spatial_chunk(eta, omega)
        special, general = (convolutions(stage, cfg, xd, dd, g) for g in (0, 1))
        for name, a, b, c in zip(("residual", "up"), special, general, rows):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b) and torch.equal(a, c), name
    finally:
        stage.close()
