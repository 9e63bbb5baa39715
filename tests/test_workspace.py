"""Device scratch of a stage and its depth (host only: a query allocates nothing).

A stage that does not keep the scratch of every residual function holds two backward
sets, whatever its depth: its workspace grows with its blocks by the two compute copies
of their conv weights and nothing else.  Small stages may keep all sets, up to 32 MiB."""
import pytest

import synth

B, F = synth.CIFAR_STAGE, synth.BLOCK_FP32
NECK = synth.IMAGENET_BOTTLENECK_STAGE
KEEP = 32 << 20

LARGE = {
    "fp32_128x32x32x32": F.with_(n=128, h=32, w=32, c_half=32),
    "fp32_256x16x16x128": F.with_(n=256, h=16, w=16, c_half=128),
    "fp32_bottleneck_64x56x56x128": NECK.with_(dtype="fp32"),
    "fp32_bottleneck_64x14x14x512": NECK.with_(n=64, h=14, w=14, c_half=512, c_mid=128, dtype="fp32"),
    "bf16_256x56x56x64": B.with_(n=256, h=56, w=56, c_half=64),
    "bf16_128x28x28x128": B.with_(n=128, h=28, w=28, c_half=128),
    "bf16_bottleneck_128x23x23x128": NECK.with_(n=128, h=23, w=23),
    "bf16_64x64x64x64": B.with_(n=64, h=64, w=64, c_half=64),
}
SMALL = {
    "fp32_8x8x8x16": F,
    "bf16_128x4x4x256": B.with_(h=4, w=4, c_half=256),
    "bf16_bottleneck_8x14x14x256": NECK.with_(n=8, h=14, w=14, c_half=256, c_mid=64),
}


def query(wl, blocks):
    """(workspace bytes, bytes of the two compute copies of the conv weights)."""
    from paper_2406_02052_amd import _lib as L
    h = L.petra_stage_create(L.StageDesc(
        wl.n, wl.h, wl.w, wl.c_half, wl.c_mid, blocks,
        L.PETRA_BLOCK_BASIC if wl.kind == "basic" else L.PETRA_BLOCK_BOTTLENECK,
        L.PETRA_BF16 if wl.dtype == "bf16" else L.PETRA_FP32, wl.bn_eps, wl.bn_momentum))
    try:
        ws = L.petra_stage_query(h)[3]
    finally:
        L.petra_stage_destroy(h)
    numel = 2 * sum(o * r * s * i for o, r, s, i in wl.conv_layers()) * blocks
    return ws, 2 * numel * (2 if wl.dtype == "bf16" else 4)


@pytest.mark.parametrize("name", list(LARGE))
def test_scratch_does_not_grow_with_depth(name):
    ws, copies = query(LARGE[name], 2)
    for blocks in (3, 6, 16):
        ws_b, copies_b = query(LARGE[name], blocks)
        assert ws_b - copies_b <= ws - copies + 1024, (blocks, ws, ws_b)   # 256-byte alignment


@pytest.mark.parametrize("name", list(SMALL))
def test_small_stages_keep_little(name):
    # beside what a stage keeps: the partial sums of its layers, which share a launch's
    # workgroups (256 of 64 x 64 channels and 9 taps, or 768 of one tap) and are at
    # least one each
    wl = SMALL[name]
    one = 256 * 64 * 64 * 9 * 4
    for blocks in (2, 6, 16):
        ws, copies = query(wl, 1)
        ws_b, copies_b = query(wl, blocks)
        assert ws_b - ws <= copies_b - copies + KEEP + max(2 * one, copies_b * 2), (blocks, ws, ws_b)
