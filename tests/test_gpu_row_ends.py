"""Launches whose rows (or image rows, whose pixels) end inside a tile: what lies behind them is neither written nor read (buffer
descriptors over what exists drop those stores and give zero for those loads). Known values lie there."""
import numpy as np
import pytest
import torch

from oracle import lightcache_oracle as lo
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import check, dev, dev32, host, make_stage, rows_to_planar

pytestmark = pytest.mark.gpu

BEHIND = 256  # rows behind the end: more than any tile's


# one row into a tile and one row short of one, on every tile of fp32 rows: 64 x 64 and 128 x 160 (320 channels), 64 x 64,
# 64 x 128 and 128 x 128 (512 channels)
@pytest.mark.parametrize("C,heads,rows", [(320, 5, 33), (320, 5, 20007), (512, 8, 63), (512, 8, 4001), (512, 8, 9001)])
def test_projection_with_residual(C, heads, rows):
    cfg = synth.StageConfig("ends", B=1, F=1, H=6, W=10, C_lat=4, C=C, C_deep=64, groups=32, n_res=0, heads=heads, head_dim=64, dtype="bf16")
    print(f"[case] {rows} rows of {C}", flush=True)
    stage, w = make_stage(cfg, seed=7)
    try:
        rng = np.random.default_rng(1)
        a = synth.round_to_bf16(rng.standard_normal((rows + BEHIND, C)).astype(np.float32))
        a[rows:] = np.nan
        r = rng.standard_normal((rows + BEHIND, C)).astype(np.float32)
        ad, rd = dev(stage, a), dev32(stage, r)
        y = torch.full_like(rd, 7.0)
        inplace = rd.clone()
        lcb.lc_op_proj(stage.ctx, lcb.LC_L_SATTN, ad.data_ptr(), rd.data_ptr(), y.data_ptr(), rows)
        lcb.lc_op_proj(stage.ctx, lcb.LC_L_SATTN, ad.data_ptr(), inplace.data_ptr(), inplace.data_ptr(), rows)
        stage.sync()
        assert bool((y[rows:] == 7.0).all()) and torch.equal(inplace[rows:], rd[rows:])
        assert torch.equal(y[:rows], inplace[:rows])
        ref = r[:rows].astype(np.float64) + a[:rows].astype(np.float64) @ w["sattn.wo"].astype(np.float64).T + w["sattn.bo"].astype(np.float64)
        check("projection", host(y[:rows]), ref, cfg.dtype, wide_range=True)
    finally:
        stage.close()


# the gated sums of a transformer block write the hidden states, behind which the cached entry lies
@pytest.mark.parametrize("B,T,D", [(1, 33, 256), (3, 85, 512)])
def test_gated_sum(B, T, D):
    cfg = synth.DITS["video_dit"].with_(B=B, T=T, D=D, heads=D // 64, L=3, cache_a=1, cache_b=2, token_chunk=0)
    dit = lcb.Dit(cfg, synth.make_dit_weights(cfg, 0), host_slots=0, dev_slots=1, token_chunk=0)
    try:
        entry = dit.to_device(synth.make_dit_hidden(cfg, 5))
        out = dit.empty(B, T, D)
        dit.cache_write(0, entry)
        dit.cached_step(dit.to_device(synth.make_dit_hidden(cfg, 1)), dit.to_device(synth.make_dit_modulation(cfg, 2)), out, 0)
        dit.sync()
        assert bool(torch.isfinite(out).all()) and torch.equal(dit.dev_entry(0), entry.reshape(dit.dev_entry(0).shape))
    finally:
        dit.close()


# image rows that end inside a 32-pixel segment: the last row of a launch's last frame, with another frame behind it
@pytest.mark.parametrize("C,H,W", [(320, 6, 34), (64, 6, 62), (128, 2, 12)])
def test_first_convolution(C, H, W):
    cfg = synth.StageConfig("ends", B=1, F=2, H=H, W=W, C_lat=4, C=C, C_deep=64, groups=32, n_res=0, heads=C // 64, head_dim=64, dtype="bf16")
    stage, w = make_stage(cfg, seed=7)
    try:
        x = synth.make_latents(cfg, 3).reshape(2, 4, H, W)
        xd = dev(stage, x)
        h = torch.full((2 * H * W, C), 7.0, dtype=torch.float32, device=stage.device)
        lcb.lc_op_conv_in(stage.ctx, xd.data_ptr(), h.data_ptr(), 1)
        stage.sync()
        assert bool((h[H * W:] == 7.0).all())
        ref = lo.conv3x3(x[:1].astype(np.float64), w["conv_in.w"].astype(np.float64), w["conv_in.b"].astype(np.float64))
        check("conv_in", rows_to_planar(host(h[:H * W]), 1, C, H, W), ref, cfg.dtype)
    finally:
        stage.close()
