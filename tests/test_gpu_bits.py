"""The bits of what the GELU layers give: a normal step of a bf16 transformer stack (GELU in the first MLP layer's epilogue) and
of a bf16 U-Net (GEGLU), as recorded. Both paths are deterministic, and tiles, chunks and kernels agree bit for bit, so
another digest means that the arithmetic of an element has changed: also where the result is as good, the roundings behind it
spread an ulp of a GELU to 1e-3 .. 1e-2 of the step's output, which a user who compares runs sees."""
import hashlib

import pytest

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth
from tests.gpu_util import host

pytestmark = pytest.mark.gpu


def digest(*tensors):
    h = hashlib.sha256()
    for t in tensors:
        h.update(host(t).tobytes())
    return h.hexdigest()[:16]


def dit_digest():
    cfg = synth.DitConfig("bits", B=2, T=96, D=256, heads=4, head_dim=64, L=2, cache_a=1, cache_b=2, dtype="bf16", mlp_ratio=4)
    dit = lcb.Dit(cfg, synth.make_dit_weights(cfg, 0), host_slots=0, dev_slots=1, token_chunk=0)
    try:
        out = dit.empty(cfg.B, cfg.T, cfg.D)
        dit.full_step(dit.to_device(synth.make_dit_hidden(cfg, 1)), dit.to_device(synth.make_dit_modulation(cfg, 2)), out, 0)
        dit.sync()
        return digest(out, dit.dev_entry(0))
    finally:
        dit.close()


def unet_digest():
    cfg = synth.UnetConfig("bits", B=1, F=8, H=32, W=32, C_lat=4, C=320, C1=320, C2=320, groups=32, head_dim=40, ctx_len=7, ctx_dim=64,
                           temb_dim=64, dtype="bf16")
    net = lcb.Unet(cfg, synth.make_unet_weights(cfg, 0), host_slots=0, dev_slots=1)
    try:
        x, temb, ctx = synth.make_unet_inputs(cfg, 1)
        eps = net.empty(*x.shape)
        net.full_step(net.to_device(x), net.to_device(temb), net.to_device(ctx), eps, 0)
        net.sync()
        return digest(eps, net.dev_entry(0))
    finally:
        net.close()


@pytest.mark.parametrize("run,recorded", [(dit_digest, "376869be64cc6887"), (unet_digest, "82ffaf109702786d")], ids=["dit", "unet"])
def test_recorded_bits(run, recorded):
    assert run() == recorded
