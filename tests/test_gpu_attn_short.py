"""Spatial attention over fewer tokens than one stage of keys (64): what lies behind the tokens in the V^T buffer is never
written, so it holds whatever the workspace held before. The steps are run in a workspace full of NaN."""
import numpy as np
import pytest
import torch

from oracle import dit_oracle as dito
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import check, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,heads", [(2, 1, 256, 4), (2, 16, 256, 4), (2, 24, 320, 8), (1, 33, 256, 4), (2, 63, 320, 8), (1, 64, 256, 4), (2, 65, 256, 4)])
def test_tokens_behind_the_sequence_are_ignored(B, T, D, heads):
    cfg = synth.DITS["video_dit"].with_(B=B, T=T, D=D, heads=heads, head_dim=D // heads, L=2, cache_a=1, cache_b=2, token_chunk=0)
    w = synth.make_dit_weights(cfg, 0)
    dit = lcb.Dit(cfg, w, host_slots=0, dev_slots=1, token_chunk=0)
    try:
        x, mod = synth.make_dit_hidden(cfg, 1), synth.make_dit_modulation(cfg, 2)
        out = dit.empty(B, T, D)
        xd, md = dit.to_device(x), dit.to_device(mod)
        dit.arena.fill_(255)  # 0xFFFF is a bf16 NaN
        torch.cuda.synchronize()
        dit.full_step(xd, md, out, 0)
        dit.sync()
        orc = dito.DitOracle(cfg, {k: v.astype(np.float64) for k, v in w.items()})
        check("normal step", host(out), orc.full_step(x, mod, 0), cfg.dtype, wide_range=True)
    finally:
        dit.close()
