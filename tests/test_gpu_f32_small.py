"""fp32 stages too small to fill the chip. Convolutions: 32 channels a workgroup in launches of few workgroups, the bits of the
wide ones."""
import pytest
import torch

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import dev32, empty32, make_stage

pytestmark = pytest.mark.gpu


def config(F, H, W, heads, d):
    C = heads * d
    return synth.StageConfig(f"small_{heads}x{d}_{H}x{W}", B=1, F=F, H=H, W=W, C_lat=4, C=C, C_deep=64, groups=8 if C == 64 else 32, n_res=1,
                             heads=heads, head_dim=d, dtype="f32")


@pytest.mark.parametrize("heads,d,F", [(1, 64, 70), (8, 40, 40)])
def test_narrow_convolutions_give_the_bits_of_wide_ones(heads, d, F):
    """16 x 16 images are two tiles a frame: all frames fill more than 128 workgroups, one frame does not."""
    cfg = config(F, 16, 16, heads, d)
    stage, _ = make_stage(cfg, seed=8)
    try:
        rows = cfg.H * cfg.W
        x = dev32(stage, synth.make_activation((cfg.N * rows, cfg.C), 3, "f32"))
        wide, narrow = empty32(stage, *x.shape), empty32(stage, rows, cfg.C)
        lcb.lc_op_res_block(stage.ctx, lcb.LC_L_RES0, x.data_ptr(), wide.data_ptr(), cfg.N)
        lcb.lc_op_res_block(stage.ctx, lcb.LC_L_RES0, x.data_ptr(), narrow.data_ptr(), 1)
        stage.sync()
        assert torch.equal(wide[:rows], narrow)
    finally:
        stage.close()
