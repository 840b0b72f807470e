"""The work that a user of this framework has it do, as cases that can be timed.

A denoising loop runs on torch's current stream; the framework's steps run on a compute stream of their own. So `run`
does what such a loop does around a step: the compute stream waits for the loop's stream (the latents come from the
sampler), the step is issued, and the loop's stream waits for the compute stream (the sampler reads what it returns).
Nothing waits on the host.

Paths, and what stands for them:
  stage      the cache-hit step of the shallow stage and one refresh interval of it (normal step, the deep feature
             swapped out to pinned host memory, cache steps with the entry prefetched one step ahead)
  decoder    sliced decoding of the latents to images
  dit        the normal and the cache step of the diffusion-transformer block stack
  unet       the normal and the cache step of the U-Net with real block internals
Weights are ~N(0, 0.02), norm scales 1 + N(0, 0.02), latents and hidden states ~N(0, 1), as in the package's own
synthetic workloads; everything is drawn on the GPU from the seed.
"""
import math

import torch

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth

# The sizes that listed cases share: a 16-frame video of 512 x 512 (64 x 64 latents) with the widths of the
# AnimateDiff-like stage, and the SVD-XT-like one.
_WIDTHS = {"C": 320, "C_deep": 640, "n_res": 2, "dtype": "bf16"}


def _stage(name, **kw):
    c = {"name": name, "path": "stage", "op": "cached", "B": 2, "frame_chunk": 0, "token_chunk": 0, "heads": 8, "head_dim": 40}
    c.update(_WIDTHS)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a float32 stage of 8 small frames, two at a time; bound by latency and launches
        _stage("stage_tiny_f32", B=1, F=8, H=32, W=32, C=64, C_deep=128, n_res=1, heads=1, head_dim=64, dtype="f32", frame_chunk=2),
        # the ordinary call: guidance pair of 16 frames of 512 x 512, feature chunk of 4 frames
        _stage("stage_512_cached", F=16, H=64, W=64, frame_chunk=4),
        # the same video over one refresh interval of 3 steps, swapped and prefetched, feature chunk of 8 frames
        _stage("stage_512_interval", op="interval", F=16, H=64, W=64, frame_chunk=8),
        # image-to-video at 1024 x 576: 25 frames (odd), heads of 64, frame and token chunks
        _stage("stage_1024_cached", F=25, H=72, W=128, heads=5, head_dim=64, frame_chunk=5, token_chunk=2304),
        # a short clip of an odd size without guidance: 480 x 288 is 60 x 36 latents, whose rows and frames fill no
        # whole tiles; 9 frames, chunk of 4 with a remainder
        _stage("stage_480x288_ragged", B=1, F=9, H=36, W=60, frame_chunk=4),
        # the largest stage: 32 frames of 768 x 768
        _stage("stage_768_cached", F=32, H=96, W=96, frame_chunk=8),
        # decoding 16 frames to 512 x 512 frame by frame, the slice the method is about
        {"name": "decode_frame_by_frame", "path": "decoder", "N": 16, "H": 64, "W": 64, "slice": 1, "dtype": "bf16"},
        # and with memory to spare: an odd number of frames of an odd size, four at a time
        {"name": "decode_four_ragged", "path": "decoder", "N": 7, "H": 40, "W": 56, "slice": 4, "dtype": "bf16"},
        # the transformer stack over all tokens of a guidance pair: the normal step
        {"name": "dit_normal", "path": "dit", "op": "full", "B": 2, "T": 4096, "D": 1024, "L": 12, "a": 2, "b": 10, "chunk": 0},
        # a cache step of it on fewer tokens (3 latent frames of 28 x 37 patches, no whole tiles), in chunks
        {"name": "dit_cached_ragged", "path": "dit", "op": "cached", "B": 2, "T": 3108, "D": 1024, "L": 12, "a": 2, "b": 10, "chunk": 1024},
        # the U-Net at 16 frames of 512 x 512: the normal step, which has every block of it
        {"name": "unet_512_normal", "path": "unet", "op": "full", "B": 2, "F": 16, "H": 64, "W": 64, "chunk": 0},
        # a cache step of it on 8 frames of 256 x 256, where launches no longer fill the chip
        {"name": "unet_256_cached", "path": "unet", "op": "cached", "B": 2, "F": 8, "H": 32, "W": 32, "chunk": 0},
    ]


def _log_between(rng, lo, hi, multiple):
    """A multiple of `multiple`, spread over the logarithm of [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / multiple)) * multiple))


def draw(rng):
    """One case of the ranges that the listed ones stand for: videos of 4..32 frames from 128 x 128 to 1024 x 768."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(("stage", "stage", "stage", "stage_f32", "decoder", "dit", "dit", "unet", "unet"))
        B = rng.choice((1, 2))
        if kind in ("stage", "stage_f32"):
            small = kind == "stage_f32"
            c = _stage("", op=rng.choice(("cached", "cached", "interval")), B=B, F=rng.randint(4, 16 if small else 32),
                       H=_log_between(rng, 16, 48 if small else 96, rng.choice((2, 8))),
                       W=_log_between(rng, 16, 48 if small else 128, rng.choice((2, 8))), frame_chunk=rng.choice((0, 2, 4, 5, 8, 16)))
            if small:
                c.update(C=64, C_deep=128, n_res=1, heads=1, head_dim=64, dtype="f32")
            else:
                c["heads"], c["head_dim"] = rng.choice(((8, 40), (8, 40), (5, 64)))
                if rng.random() < 0.25:
                    c["token_chunk"] = c["H"] * c["W"] // 4
            del c["name"]
        elif kind == "decoder":
            c = {"path": "decoder", "N": rng.randint(1, 16), "H": _log_between(rng, 16, 72, rng.choice((2, 8))),
                 "W": _log_between(rng, 16, 72, rng.choice((2, 8))), "slice": rng.choice((1, 1, 2, 4)), "dtype": "bf16"}
        elif kind == "dit":
            c = {"path": "dit", "op": rng.choice(("full", "cached")), "B": B, "T": _log_between(rng, 256, 4608, rng.choice((1, 64))),
                 "D": rng.choice((512, 768, 1024)), "L": 12, "a": 2, "b": 10, "chunk": rng.choice((0, 0, 512, 1024))}
        else:
            c = {"path": "unet", "op": rng.choice(("full", "cached")), "B": B, "F": rng.randint(4, 16),
                 "H": _log_between(rng, 16, 64, rng.choice((4, 8))), "W": _log_between(rng, 16, 64, rng.choice((4, 8))),
                 "chunk": rng.choice((0, 0, 4, 8))}
        if work(c)["flops"] <= most:
            return c


# ---- shapes ------------------------------------------------------------------------------------------------
def _config(case):
    p = case["path"]
    if p == "stage":
        return synth.StageConfig("case", case["B"], case["F"], case["H"], case["W"], 4, case["C"], case["C_deep"], 32, case["n_res"],
                                 case["heads"], case["head_dim"], case["dtype"], case["frame_chunk"], case["token_chunk"])
    if p == "decoder":
        return synth.DECODERS["animatediff"].with_(N=case["N"], H=case["H"], W=case["W"], dtype=case["dtype"])
    if p == "dit":
        return synth.DITS["video_dit"].with_(B=case["B"], T=case["T"], D=case["D"], heads=case["D"] // 64, L=case["L"],
                                             cache_a=case["a"], cache_b=case["b"], token_chunk=case["chunk"])
    return synth.UNETS["sd15_video"].with_(B=case["B"], F=case["F"], H=case["H"], W=case["W"])


def _manifest(case, cfg):
    return {"stage": synth.weight_manifest, "decoder": synth.decoder_weight_manifest, "dit": synth.dit_weight_manifest,
            "unet": synth.unet_weight_manifest}[case["path"]](cfg)


def _weights(case, cfg, gen):
    """name -> float32 array, in the manifest's order: drawn on the GPU in one go, then brought to the host, where the
    framework takes its weights from."""
    entries = _manifest(case, cfg)
    total = sum(math.prod(shape) for _, shape, _ in entries)
    flat = (torch.randn(total, generator=gen, device="cuda") * 0.02).cpu().numpy()
    out, at = {}, 0
    for name, shape, kind in entries:
        n = math.prod(shape)
        a = flat[at:at + n].reshape(shape)
        out[name] = a + 1.0 if kind == "g" else a
        at += n
    return out


def _randn(gen, shape, dtype=torch.float32):
    return torch.randn(shape, generator=gen, device="cuda").to(dtype)


def _slot_view(peek, ctx, owner, slot, shape):
    """The float32 entry in a device slot as a tensor over the holder's workspace."""
    ptr, n = peek(ctx, slot)
    off = ptr - owner.arena.data_ptr()
    return owner.arena[off:off + n].view(torch.float32).reshape(shape)


# ---- states ------------------------------------------------------------------------------------------------
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    cfg = _config(case)
    w = _weights(case, cfg, gen)
    s = {"case": dict(case)}
    if case["path"] == "stage":
        swapped = case["op"] == "interval"
        m = lcb.Stage(cfg, w, host_slots=1 if swapped else 0, dev_slots=2 if swapped else 1)
        s["x"] = _randn(gen, (cfg.B, cfg.F, cfg.C_lat, cfg.H, cfg.W), m.tdtype)
        deep = _randn(gen, (cfg.N, cfg.C_deep, cfg.H // 2, cfg.W // 2), m.tdtype)
        s["eps"] = [torch.empty_like(s["x"]) for _ in range(3 if swapped else 1)]
        if swapped:
            # the latents of the interval's steps: each a little further down the schedule
            s["xs"] = [s["x"], (s["x"] * 0.98).contiguous(), (s["x"] * 0.96).contiguous()]
        torch.cuda.synchronize()
        m.cache_write(0, deep)
        m.sync()
    elif case["path"] == "decoder":
        m = lcb.Decoder(cfg, w, max_slice=case["slice"])
        s["z"] = _randn(gen, (cfg.N, cfg.C_lat, cfg.H, cfg.W), m.tdtype)
    elif case["path"] == "dit":
        m = lcb.Dit(cfg, w, host_slots=0, dev_slots=1)
        s["x"] = _randn(gen, (cfg.B, cfg.T, cfg.D))
        s["mod"] = _randn(gen, (cfg.L, cfg.B, 6, cfg.D)) * 0.1
        s["mod"][:, :, 2] += 1.0
        s["mod"][:, :, 5] += 1.0
        s["out"] = torch.empty_like(s["x"])
        delta = _randn(gen, (cfg.B, cfg.T, cfg.D))
        torch.cuda.synchronize()
        m.cache_write(0, delta)
        m.sync()
        s["entry"] = _slot_view(lcb.lc_dit_cache_dev_peek, m.ctx, m, 0, (cfg.B, cfg.T, cfg.D))
    else:
        m = lcb.Unet(cfg, w, host_slots=0, dev_slots=1, frame_chunk=case["chunk"] or None)
        s["x"] = _randn(gen, (cfg.B, cfg.F, cfg.C_lat, cfg.H, cfg.W), m.tdtype)
        s["temb"] = _randn(gen, (cfg.B, cfg.temb_dim), m.tdtype)
        s["cond"] = _randn(gen, (cfg.B, cfg.ctx_len, cfg.ctx_dim), m.tdtype)
        s["eps"] = torch.empty_like(s["x"])
        deep = _randn(gen, (cfg.N, cfg.H * cfg.W, cfg.C1))
        torch.cuda.synchronize()
        m.cache_write(0, deep)
        m.sync()
        s["entry"] = _slot_view(lcb.lc_unet_cache_dev_peek, m.ctx, m, 0, (cfg.N, cfg.H * cfg.W, cfg.C1))
    s["m"] = m
    return s


def run(state):
    m, case = state["m"], state["case"]
    loop = torch.cuda.current_stream()
    mine = m.stream if case["path"] == "decoder" else m.compute
    mine.wait_stream(loop)
    if case["path"] == "stage":
        if case["op"] == "cached":
            m.cached_step(state["x"], state["eps"][0], 0)
            out = state["eps"][0]
        else:
            xs, eps = state["xs"], state["eps"]
            m.full_step(xs[0], eps[0], 0)
            m.swap_out(0, 0)
            m.swap_in(0, 1)  # prefetch for the next step
            m.cached_step(xs[1], eps[1], 1)
            m.swap_in(0, 0)
            m.cached_step(xs[2], eps[2], 0)
            out = eps
    elif case["path"] == "decoder":
        out = m.decode(state["z"], case["slice"])
    elif case["path"] == "dit":
        if case["op"] == "full":
            m.full_step(state["x"], state["mod"], state["out"], 0)
            out = [state["out"], state["entry"]]
        else:
            m.cached_step(state["x"], state["mod"], state["out"], 0)
            out = state["out"]
    elif case["op"] == "full":
        m.full_step(state["x"], state["temb"], state["cond"], state["eps"], 0)
        out = [state["eps"], state["entry"]]
    else:
        m.cached_step(state["x"], state["temb"], state["cond"], state["eps"], 0)
        out = state["eps"]
    loop.wait_stream(mine)
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------------
def work(case):
    """FLOPs of the contractions (the configurations' own formulas), and each input, weight and output once. Inside a
    step every map between two operators that need whole-frame statistics or all tokens could at best stay on the
    chip, so only what crosses the boundary is counted."""
    cfg = _config(case)
    es = 2 if getattr(cfg, "dtype", "bf16") == "bf16" else 4
    weights = es * sum(math.prod(shape) for _, shape, _ in _manifest(case, cfg))
    if case["path"] == "stage":
        lat = es * cfg.N * cfg.C_lat * cfg.T
        deep = es * cfg.N * cfg.C_deep * cfg.T // 4
        cached = cfg.cached_step_flops()
        if case["op"] == "cached":
            return {"bytes": weights + 2 * lat + deep, "flops": cached}
        q = cfg.N * cfg.T // 4
        full = cached + 2.0 * 9 * cfg.C * cfg.C_deep * q + 2.0 * 9 * cfg.C_deep * cfg.C_deep * q
        # the weights and latents of three steps; the entry written, copied out, brought back twice and read twice
        return {"bytes": 3 * (weights + 2 * lat) + 6 * deep, "flops": full + 2 * cached}
    if case["path"] == "decoder":
        img = es * cfg.N * cfg.C_img * cfg.H * cfg.W * 4 ** cfg.levels
        return {"bytes": weights + es * cfg.N * cfg.C_lat * cfg.H * cfg.W + img, "flops": cfg.decode_flops()}
    if case["path"] == "dit":
        hidden = 4 * cfg.B * cfg.T * cfg.D
        mod = 4 * cfg.L * cfg.B * 6 * cfg.D
        full = case["op"] == "full"
        share = 1.0 if full else (cfg.L - (cfg.cache_b - cfg.cache_a)) / cfg.L
        return {"bytes": 3 * hidden + share * (weights + mod), "flops": cfg.full_step_flops() if full else cfg.cached_step_flops()}
    lat = es * cfg.N * cfg.C_lat * cfg.H * cfg.W
    entry = 4 * cfg.N * cfg.H * cfg.W * cfg.C1
    if case["op"] == "full":
        return {"bytes": weights + 2 * lat + entry, "flops": cfg.full_step_flops()}
    deep_only = ("d0.down", "d1.", "mid.", "u2.", "u1.")
    shallow = es * sum(math.prod(shape) for name, shape, _ in _manifest(case, cfg) if not name.startswith(deep_only))
    return {"bytes": shallow + 2 * lat + entry, "flops": cfg.cached_step_flops()}


def tolerance(case):
    """What the same steps in 64 bits (the oracle) differ by, times about four: float32 stages 1e-6; bf16 operands with
    float32 sums 4.5e-3 for the stage, 3e-3 for the decoder and the transformer stack, 6.5e-3 for the U-Net, whose
    normal step is some 80 contractions deep."""
    if case["path"] == "stage" and case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 2.4e-2 if case["path"] == "unet" else 1.6e-2 if case["path"] == "stage" else 1.2e-2}
