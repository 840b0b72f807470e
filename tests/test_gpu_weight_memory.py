"""Device memory that loaded weights hold. The 3x3 weights, nearly all of it, are kept in one order that every kernel of a dtype
reads; the projections of the stage's attention blocks in two. Measured around the call that loads them, on a second holder
(the first one's call also loads the kernels)."""
import math

import pytest
import torch

from paper_2510_05367_amd import binding as lcb
from paper_2510_05367_amd import synth

pytestmark = pytest.mark.gpu

SLACK = 6 << 20  # padding of the 256-byte pieces, biases and norms held in fp32, the allocator's granularity (2 MiB a piece)


def held(monkeypatch, name, make):
    original, sizes = getattr(lcb, name), []

    def spy(*args):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        original(*args)
        torch.cuda.synchronize()
        sizes.append(before - torch.cuda.mem_get_info()[0])
    monkeypatch.setattr(lcb, name, spy)
    holders = [make(), make()]
    for h in holders:
        h.close()
    return sizes[1]


def bounds(manifest, es=2):
    conv = sum(es * math.prod(shape) for _, shape, _ in manifest if len(shape) == 4)
    rest = sum(es * math.prod(shape) for _, shape, _ in manifest if len(shape) != 4)
    return conv, rest


def case(path):
    if path == "stage":
        cfg = synth.StageConfig("mem", B=1, F=1, H=8, W=16, C_lat=4, C=640, C_deep=640, groups=32, n_res=2, heads=10, head_dim=64, dtype="bf16")
        w = synth.make_weights(cfg, 0)
        return "lc_load_weights", lambda: lcb.Stage(cfg, w, host_slots=0, dev_slots=1), bounds(synth.weight_manifest(cfg))
    if path == "decoder":
        cfg = synth.DECODERS["animatediff"].with_(N=1, H=8, W=16, widths=(640, 640, 640, 640), heads=10, head_dim=64)
        w = synth.make_decoder_weights(cfg, 0)
        return "lc_decoder_load_weights", lambda: lcb.Decoder(cfg, w), bounds(synth.decoder_weight_manifest(cfg))
    cfg = synth.UnetConfig("mem", B=1, F=1, H=8, W=16, C_lat=4, C=320, C1=640, C2=640, groups=32, head_dim=40, ctx_len=7, ctx_dim=64,
                           temb_dim=64, dtype="bf16")
    w = synth.make_unet_weights(cfg, 0)
    return "lc_unet_load_weights", lambda: lcb.Unet(cfg, w, host_slots=0, dev_slots=1), bounds(synth.unet_weight_manifest(cfg))


@pytest.mark.parametrize("path", ["stage", "decoder", "unet"])
def test_one_copy_of_the_convolutions(path, monkeypatch):
    name, make, (conv, rest) = case(path)
    n = held(monkeypatch, name, make)
    print(f"\n[{path}] 3x3 weights {conv / 2**20:.1f} MiB, others {rest / 2**20:.1f} MiB, held {n / 2**20:.1f} MiB", flush=True)
    # the measurement sees the memory, less what the runtime had left over of earlier holders' or gives back meanwhile, in pieces
    # of 2 MiB: 172 MiB for the U-Net's 171.0 alone, 170 behind the other tests of a process
    assert n >= conv + rest - SLACK
    assert n <= conv + 2 * rest + SLACK
