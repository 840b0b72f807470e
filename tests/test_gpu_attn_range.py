"""Spatial and cross-attention of the bf16 stages with scores far outside the range where nothing has to be subtracted
in the exponent: far above and below zero, leaping in a late stage of keys, climbing from stage to stage, and values so
large that only the exact maximum keeps the sums finite. In every launch ordinary queries share wavefronts with the others.
Compared with the definition in float64; a window of queries must give the bits of the whole launch; and scores of several
hundred must not cost much more time than ordinary ones."""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import lightcache_oracle as lo
from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import dev, host, make_stage, rel_l2

pytestmark = pytest.mark.gpu

KINDS = ["up", "down", "leap", "climb", "large values"]


def make_qkv(kind, N, Tq, Tk, heads, d, seed):
    """q [N][Tq], k and v [N][Tk] rows of heads * d, q in log2 units (the scale of the scores already on it)."""
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((N, Tq, heads, d)).astype(np.float32) * np.float32(2.0 / math.sqrt(d))
    k = rng.standard_normal((N, Tk, heads, d)).astype(np.float32)
    v = rng.standard_normal((N, Tk, heads, d)).astype(np.float32)
    t = np.arange(Tk)
    if kind == "up":
        q[:, ::3] *= np.float32(120.0)
    elif kind == "down":
        k[..., 0] = 4.0
        q[:, ::3, :, 0] = -60.0
    elif kind == "leap":
        k[..., 0] = 0.0
        k[:, Tk * 3 // 4, :, 0] = 10.0
        q[:, ::5, :, 0] = 15.0
    elif kind == "climb":
        k[..., 0] = (4 * (t // 32))[None, :, None]
        q[:, ::4, :, 0] = 13.0
        q[:, 1::4, :, 0] = -13.0
    else:
        k[..., 0] = np.where(t < 32, 0.0, 5.0)[None, :, None]
        q[:, ::3, :, 0] = 14.0
        v *= np.float32(2.0 ** 100)
    return tuple(synth.round_to_bf16(a.reshape(a.shape[0], a.shape[1], heads * d)) for a in (q, k, v))


def reference(q, k, v, heads, d, prescaled):
    q = q.astype(np.float64)
    if prescaled:
        q = q * (math.sqrt(d) / math.log2(math.e))
    return lo.attention_core(q, k.astype(np.float64), v.astype(np.float64), heads)


def compare(name, got, ref, vmax):
    """Roundings to bf16, 2^-9 relative each: of a probability (the denominator sums them as rounded) and of the output, so
    rel-L2 well below 1e-2. One element is a mean of values, weighted with probabilities that are off by 2^-9 in the
    numerator and in the denominator: at most 2 * 2^-9 max|v|, and 2^-9 |out| <= 2^-9 max|v| for the store."""
    assert np.all(np.isfinite(got)), f"{name}: non-finite values"
    r, m = rel_l2(got, ref), float(np.max(np.abs(got - ref)))
    print(f"{name}: rel-L2 {r:.3e}, max {m / vmax:.3e} of the largest value", flush=True)
    assert r <= 1e-2 and m <= 3 * 2.0 ** -9 * vmax, name


def stage_of(F, H, W, heads, d):
    C = heads * d
    cfg = synth.StageConfig(f"ar_{heads}x{d}", B=1, F=F, H=H, W=W, C_lat=4, C=C, C_deep=64, groups=8 if C == 64 else 32, n_res=1,
                            heads=heads, head_dim=d, dtype="bf16")
    return make_stage(cfg, seed=6)[0], cfg


@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads,d,F,H,W", [(8, 8, 2, 10, 14), (4, 16, 2, 10, 14), (2, 32, 2, 10, 14), (8, 40, 2, 10, 14), (5, 64, 2, 10, 14),
                                           (8, 40, 16, 18, 30), (5, 64, 18, 18, 30)])
def test_spatial_attention_far_scores(heads, d, F, H, W, kind, prescaled):
    stage, cfg = stage_of(F, H, W, heads, d)
    try:
        N, T, C = cfg.N, cfg.T, cfg.C
        q, k, v = make_qkv(kind, N, T, T, heads, d, 91)
        if not prescaled:
            q = synth.round_to_bf16(q * np.float32(math.sqrt(d) / math.log2(math.e)))
        qd = dev(stage, np.concatenate([q, k, v], axis=2).reshape(N * T, 3 * C))
        out = stage.empty(N * T, C)
        lcb.lc_op_spatial_attention(stage.ctx, qd.data_ptr(), out.data_ptr(), N, 0, T, prescaled)
        part = stage.empty(N * T, C)
        part.copy_(out)
        part.view(N, T, C)[:, 7:61].fill_(3.0)
        lcb.lc_op_spatial_attention(stage.ctx, qd.data_ptr(), part.data_ptr(), N, 7, 61, prescaled)
        stage.sync()
        n = min(N, 3)  # (the frames are alike)
        compare(f"spatial {heads}x{d} T={T} {kind} prescaled={prescaled}", host(out).reshape(N, T, C)[:n],
                reference(q[:n], k[:n], v[:n], heads, d, prescaled), float(np.max(np.abs(v))))
        assert torch.equal(out, part)
    finally:
        stage.close()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads,d,frames,kv_div,Tq,Tk", [(8, 40, 4, 2, 140, 77), (5, 64, 4, 4, 140, 77), (4, 16, 2, 1, 33, 200), (8, 40, 24, 12, 300, 77),
                                                         (5, 64, 20, 10, 530, 77)])
def test_cross_attention_far_scores(heads, d, frames, kv_div, Tq, Tk, kind):
    """The launcher itself: the U-Net's layers around it would turn the rounding of such peaked scores into other outputs."""
    lib, P, I = lcb.lib(), ctypes.c_void_p, ctypes.c_int
    cross = getattr(lib, "_ZN2lc22launch_cross_attentionEP12ihipStream_tiPKviS3_iS3_iPviiiiii")
    cross.restype, cross.argtypes = I, [P, I, P, I, P, I, P, I, P, I, I, I, I, I, I]
    make_vt = getattr(lib, "_ZN2lc14launch_make_vtEP12ihipStream_tiPKviPviiii")
    make_vt.restype, make_vt.argtypes = I, [P, I, P, I, P, I, I, I, I]
    C, G, Tp = heads * d, frames // kv_div, (Tk + 63) // 64 * 64
    q, k, v = make_qkv(kind, frames, Tq, Tk, heads, d, 92)
    k, v = k[:G], v[:G]
    on = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16)
    qd, kd, vd = on(q), on(k), on(v)
    vt = torch.full((G, C, Tp), float("nan"), device="cuda", dtype=torch.bfloat16)  # (what lies behind the keys is not trusted)
    out = torch.empty(frames, Tq, C, device="cuda", dtype=torch.bfloat16)
    s = torch.cuda.current_stream().cuda_stream
    assert make_vt(s, lcb.LC_BF16, vd.data_ptr(), C, vt.data_ptr(), G, Tk, Tp, C) == 0
    assert cross(s, lcb.LC_BF16, qd.data_ptr(), C, kd.data_ptr(), C, vt.data_ptr(), Tp, out.data_ptr(), frames, Tq, Tk, kv_div, heads, d) == 0
    torch.cuda.synchronize()
    n = np.arange(0, frames, max(1, frames // 3))
    compare(f"cross {heads}x{d} Tk={Tk} {kind}", host(out)[n], reference(q[n], k[n // kv_div], v[n // kv_div], heads, d, 1),
            float(np.max(np.abs(v))))


@pytest.mark.parametrize("heads,d", [(8, 40), (5, 64)])
def test_far_scores_cost_little_more(heads, d):
    """Scores with a deviation of 150 and 500 and scores 240 below zero, in log2 units, against ordinary ones: one sweep over
    the keys with a subtraction per score and some rescaling (1.1 to 1.4 times as long), not two or three sweeps (2.4)."""
    stage, cfg = stage_of(4, 64, 64, heads, d)
    try:
        N, T, C = cfg.N, cfg.T, cfg.C
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        x = torch.randn(N, T, 3, heads, d, generator=g, device="cuda")
        out = stage.empty(N * T, C)

        def us(qkv):
            rows = qkv.reshape(N * T, 3 * C).to(torch.bfloat16).contiguous()
            best = float("inf")
            for _ in range(6):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(10):
                    lcb.lc_op_spatial_attention(stage.ctx, rows.data_ptr(), out.data_ptr(), N, 0, T, 1)
                b.record()
                torch.cuda.synchronize()
                best = min(best, a.elapsed_time(b) * 100)
            return best

        def scaled(std):
            y = x.clone()
            y[:, :, 0] *= std / math.sqrt(d)
            return y

        down = scaled(2.0)
        down[:, :, 1, :, 0] = 4.0
        down[:, :, 0, :, 0] = -60.0
        base = us(scaled(2.0))
        for name, y in (("150", scaled(150.0)), ("500", scaled(500.0)), ("-240", down)):
            t = us(y)
            print(f"{heads}x{d}: ordinary {base:.0f} us, {name}: {t:.0f} us", flush=True)
            assert t < 1.8 * base, (name, t, base)
    finally:
        stage.close()
