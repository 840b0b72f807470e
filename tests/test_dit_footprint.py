"""The footprint that the transformer stack states, against what its passes use (host only)."""
from paper_2510_05367_amd import binding as lcb
from tests.test_gpu_dit import BIG, TWO_APART, TWO_F32, TWO_GATED, mlp_passes


def test_workspace_holds_nothing_that_no_pass_uses():
    """The MLP of the benchmark's stack needs no more than attention held, with or without a chunk; where it does, the workspace
    without a chunk is what one pass takes."""
    big = lcb.make_dit_config(BIG, 0, 1)
    R, D = BIG.B * BIG.T, BIG.D
    need = 2 * R * D * 4 + 10 * R * D  # hidden states and one entry; q,k,v, V^T and attention output
    for chunk in (0, 1, 1024):
        assert lcb.lc_dit_workspace_bytes(big, chunk) == need, chunk
        assert mlp_passes(BIG, chunk)[0] == 1
    for cfg in (TWO_GATED, TWO_APART, TWO_F32):
        passes, rows = mlp_passes(cfg, 0)
        assert passes == 1 and rows == cfg.B * cfg.T
        for chunk in (1, 16, 64, cfg.B * cfg.T - 1):
            assert lcb.lc_dit_workspace_bytes(lcb.make_dit_config(cfg, 0, 1), chunk) <= lcb.lc_dit_workspace_bytes(lcb.make_dit_config(cfg, 0, 1), 0)
