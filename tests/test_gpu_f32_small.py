"""fp32 stages too small to fill the chip. Spatial attention: four wavefronts share their queries and split the keys (stages of
128 keys, 32 a wavefront), so sequences that leave wavefronts without keys, or end inside one's; scores that leap far up in one
wavefront's keys only. Convolutions: 32 channels a workgroup in launches of few workgroups, the bits of the wide ones."""
import numpy as np
import pytest
import torch

from oracle import lightcache_oracle as lo
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import check, dev, dev32, empty32, host, make_stage

pytestmark = pytest.mark.gpu


def config(F, H, W, heads, d):
    C = heads * d
    return synth.StageConfig(f"small_{heads}x{d}_{H}x{W}", B=1, F=F, H=H, W=W, C_lat=4, C=C, C_deep=64, groups=8 if C == 64 else 32, n_res=1,
                             heads=heads, head_dim=d, dtype="f32")


# T = 64 (not split), 72 (a sub-tile of 8 keys, two wavefronts with none), 100, 128, 140 (a second stage of 12), 288, 1024; the last
# has 18 x 8 x 2 blocks of 128 queries: not split
@pytest.mark.parametrize("heads,d,F,H,W", [(1, 64, 2, 4, 16), (1, 64, 2, 6, 12), (8, 8, 2, 10, 10), (4, 16, 2, 8, 16), (2, 32, 2, 10, 14), (8, 40, 2, 16, 18),
                                           (1, 64, 3, 32, 32), (8, 40, 18, 10, 14)])
@pytest.mark.parametrize("kind", ["plain", "leap"])
def test_spatial_attention(heads, d, F, H, W, kind):
    cfg = config(F, H, W, heads, d)
    stage, _ = make_stage(cfg, seed=6)
    try:
        N, T, C = cfg.N, cfg.T, cfg.C
        rng = np.random.default_rng(7)
        q, k, v = (rng.standard_normal((N, T, heads, d)).astype(np.float32) for _ in range(3))
        if kind == "leap":  # one late key far above the others for some queries, all keys of one wavefront far below for others
            q[:, ::5, :, 0], k[..., 0] = 12.0, 0.0
            k[:, T * 3 // 4, :, 0] = 8.0
            k[:, 32:64, :, 1], q[:, 1::5, :, 1] = -20.0, 6.0
        q, k, v = (a.reshape(N, T, C) for a in (q, k, v))
        qd = dev(stage, np.concatenate([q, k, v], axis=2).reshape(N * T, 3 * C))
        out = stage.empty(N * T, C)
        lcb.lc_op_spatial_attention(stage.ctx, qd.data_ptr(), out.data_ptr(), N, 0, T, 0)
        part, one = out.clone(), out.clone()
        part.view(N, T, C)[:, 7:61].fill_(3.0)
        one[:T].fill_(3.0)
        lcb.lc_op_spatial_attention(stage.ctx, qd.data_ptr(), part.data_ptr(), N, 7, 61, 0)  # a range of queries
        lcb.lc_op_spatial_attention(stage.ctx, qd.data_ptr(), one.data_ptr(), 1, 0, T, 0)    # a chunk of frames
        stage.sync()
        n = min(N, 3)
        check(f"attention {cfg.name} {kind}", host(out).reshape(N, T, C)[:n],
              lo.attention_core(q[:n].astype(np.float64), k[:n].astype(np.float64), v[:n].astype(np.float64), heads), "f32")
        assert torch.equal(out, part) and torch.equal(out, one)
    finally:
        stage.close()


# the split where its workgroups of 32 queries are at most one per compute unit, or the sequence is long, or the problems (heads x
# frames) are a multiple of eight: on either side of each. A stage of 200 frames never splits; its operator on the first F of
# them gives the bits of a stage of F that does not, and others (of the same result) than one that does
@pytest.mark.parametrize("heads,d,F,H,W,split", [(5, 64, 25, 8, 16, False), (5, 64, 12, 8, 16, True), (5, 64, 16, 8, 16, True), (5, 64, 9, 12, 16, False),
                                                 (5, 64, 9, 14, 16, True), (8, 40, 15, 8, 16, True), (3, 64, 22, 8, 16, False)])
def test_split_keys_where_they_pay(heads, d, F, H, W, split):
    cfg = config(F, H, W, heads, d)
    few, many = make_stage(cfg, seed=6)[0], make_stage(cfg.with_(F=200), seed=6)[0]
    try:
        rng = np.random.default_rng(7)
        qd = dev(few, rng.standard_normal((F * cfg.T, 3 * cfg.C)).astype(np.float32))
        outs = []
        for st in (few, many):
            outs.append(st.empty(F * cfg.T, cfg.C))
            torch.cuda.synchronize()
            lcb.lc_op_spatial_attention(st.ctx, qd.data_ptr(), outs[-1].data_ptr(), F, 0, cfg.T, 0)
            st.sync()
        assert torch.equal(*outs) == (not split)
        assert float((outs[0] - outs[1]).norm() / outs[1].norm()) < 1e-5
    finally:
        few.close()
        many.close()


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
