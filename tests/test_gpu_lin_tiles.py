"""The tiles a dense linear layer may take by its number of rows (lc_lin3.hip): every output element is contracted in the
same order by all of them, so a transformer step on a few batch elements, which takes the small tiles, has to give the bits
of the step on all of them at once, which takes the large ones (which tiles these are: test_lin_dispatch.py); with the gated
sum in the projections' epilogues over rows of several batch elements, V^T from the projection's epilogue (rows in fours) and
from its own pass (odd token counts). A token chunk does not reach other tiles, since the MLP of these stacks has room for
all rows whatever the chunk; it must not change a bit either."""
import numpy as np
import pytest
import torch

from oracle import dit_oracle as dito
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import check, host

pytestmark = pytest.mark.gpu

BASE = synth.DITS["video_dit"]


def steps(cfg, dit, xd, md):
    full, cached = dit.empty(cfg.B, cfg.T, cfg.D), dit.empty(cfg.B, cfg.T, cfg.D)
    dit.full_step(xd, md, full, 0)
    dit.cached_step(xd, md, cached, 0)
    dit.sync()
    return full, cached, dit.dev_entry(0).clone()


# B, T, D, heads, batch elements at a time: all at once 256 x 256 (MLP, 4092 rows of 1024), 256 x 192 (q,k,v) and 64 x 128 tiles, four
# at a time 64 x 128 and 64 x 64, one 64 x 64; 128 x 128 with an odd token count (no fused V^T) against small tiles; widths of
# 160 channels: 128 x 160 (q,k,v, MLP) against 64 x 64. Every one with a remainder of rows
SPLITS = [(33, 124, 1024, 16, (4, 1)), (24, 129, 1024, 16, (5, 1)), (33, 124, 640, 10, (8, 1))]


@pytest.mark.parametrize("B,T,D,heads,groups", SPLITS)
def test_batch_elements_alone_give_the_bits_of_all(B, T, D, heads, groups):
    cfg = BASE.with_(B=B, T=T, D=D, heads=heads, L=2, cache_a=1, cache_b=2, token_chunk=0)
    w = synth.make_dit_weights(cfg, 0)
    x, mod = synth.make_dit_hidden(cfg, 1), synth.make_dit_modulation(cfg, 2)

    def run(c, xs, ms):
        dit = lcb.Dit(c, w, host_slots=0, dev_slots=1, token_chunk=0)
        try:
            return steps(c, dit, dit.to_device(np.ascontiguousarray(xs)), dit.to_device(np.ascontiguousarray(ms)))
        finally:
            dit.close()
    ref = run(cfg, x, mod)
    assert bool(torch.isfinite(ref[0]).all()) and torch.equal(ref[0], ref[1])
    for n in groups:
        for b in sorted({0, (B // n) // 2 * n, B - n}):  # the first ones, some in the middle and the last, whose rows end the matrix
            print(f"[case] {B} x {T} x {D}: batch elements {b}..{b + n - 1}", flush=True)
            got = run(cfg.with_(B=n), x[b:b + n], mod[:, b:b + n])
            for name, g, r in zip(("normal step", "cache step", "Delta"), got, ref):
                assert torch.equal(g.reshape(n, T, D), r.reshape(B, T, D)[b:b + n]), (name, n, b)


# rows x width: 256 x 256, 256 x 192 and 128 x 128 tiles; a remainder of rows in every tile; an odd token
# count (no fused V^T); widths that the 192-channel tile does not divide
@pytest.mark.parametrize("B,T,D,chunks", [(2, 2048, 1024, (1024, 388)), (1, 8190, 512, (2000, 61)), (3, 1363, 768, (640, 1000)), (2, 129, 1024, (64, 7))])
def test_tiles_agree_bitwise(B, T, D, chunks):
    cfg = BASE.with_(B=B, T=T, D=D, heads=D // 64, L=2, cache_a=1, cache_b=2, token_chunk=0)
    dit = lcb.Dit(cfg, synth.make_dit_weights(cfg, 0), host_slots=0, dev_slots=1, token_chunk=0)
    try:
        xd, md = dit.to_device(synth.make_dit_hidden(cfg, 1)), dit.to_device(synth.make_dit_modulation(cfg, 2))
        ref = steps(cfg, dit, xd, md)
        assert bool(torch.isfinite(ref[0]).all()) and torch.equal(ref[0], ref[1])
        for chunk in chunks:
            print(f"[case] {B} x {T} x {D} chunk {chunk}", flush=True)
            dit.set_chunk(chunk)
            for a, b in zip(steps(cfg, dit, xd, md), ref):
                assert torch.equal(a, b), chunk
    finally:
        dit.close()


# gate vectors that change inside a 32-row tile (T = 36, 33), one row beyond a tile, fewer tokens than the fused sum takes
@pytest.mark.parametrize("B,T,D", [(4, 36, 512), (3, 33, 256), (2, 65, 384), (2, 24, 256)])
def test_gated_epilogue_matches_oracle(B, T, D):
    cfg = BASE.with_(B=B, T=T, D=D, heads=D // 64, L=2, cache_a=1, cache_b=2, token_chunk=0)
    w = synth.make_dit_weights(cfg, 0)  # (flat softmax: a peaked one turns the rounding of a score into a change of the output
    # that has nothing to do with the sum tested here; with logits of std 8 two bf16 attention kernels differ by 0.026 at 4 x 36 x 512)
    dit = lcb.Dit(cfg, w, host_slots=0, dev_slots=1, token_chunk=0)
    try:
        x, mod = synth.make_dit_hidden(cfg, 1), synth.make_dit_modulation(cfg, 2)
        full, cached, delta = steps(cfg, dit, dit.to_device(x), dit.to_device(mod))
        orc = dito.DitOracle(cfg, {k: v.astype(np.float64) for k, v in w.items()})
        check("normal step", host(full), orc.full_step(x, mod, 0), cfg.dtype, wide_range=True)
        check("Delta", host(delta), orc.dev[0], cfg.dtype)
        assert torch.equal(cached, full)
    finally:
        dit.close()


# exactly 256 tiles of 128 x 128, and one row more (width 1024); widths of 160-channel tiles, exactly 128 of them and one row more
@pytest.mark.parametrize("T,D,heads,chunk", [(4096, 1024, 16, 640), (4097, 1024, 16, 640), (4096, 640, 10, 1000), (4097, 640, 10, 1000)])
def test_tiles_agree_bitwise_at_the_lines_between_them(T, D, heads, chunk):
    cfg = BASE.with_(B=1, T=T, D=D, heads=heads, L=2, cache_a=1, cache_b=2, token_chunk=0)
    dit = lcb.Dit(cfg, synth.make_dit_weights(cfg, 0), host_slots=0, dev_slots=1, token_chunk=0)
    try:
        xd, md = dit.to_device(synth.make_dit_hidden(cfg, 1)), dit.to_device(synth.make_dit_modulation(cfg, 2))
        ref = steps(cfg, dit, xd, md)
        assert bool(torch.isfinite(ref[0]).all()) and torch.equal(ref[0], ref[1])
        dit.set_chunk(chunk)
        for a, b in zip(steps(cfg, dit, xd, md), ref):
            assert torch.equal(a, b)
    finally:
        dit.close()
