"""GPU parity of the convolutions and weight gradients on flattened pixels, at the
edges of their tiles and of the rules that choose between them (the bars of
tests/harness.py, without the direction anchor: that one compares the oracle's bf16
storage model with plain fp64, which over as few rows as here, 126 in the smallest
case, are 0.978 apart by themselves in a BN beta the GPU has to 1.7e-5)."""
import pytest

import synth
from tests.harness import check, gpu_stage, run_step_parity

pytestmark = pytest.mark.gpu

B, F = synth.CIFAR_STAGE, synth.BLOCK_FP32
NECK = synth.IMAGENET_BOTTLENECK_STAGE

CASES = {
    # one padded chunk (c = 16); a single column; 65 pixels: one past a tile
    "bf16_c16_70x1x1": B.with_(n=70, h=1, w=1, c_half=16, blocks=1),
    "bf16_c32_2x33x1": B.with_(n=2, h=33, w=1, blocks=1),
    "bf16_c64_1x13x5": B.with_(n=1, h=13, w=5, c_half=64, blocks=1),
    # the 128-pixel tile: the smallest size that takes it, its last tile ragged
    "bf16_c32_1x233x141": B.with_(n=1, h=233, w=141, blocks=1),
    # four K waves: the widest image whose patches fit and the next one; two and
    # four chunks per wave
    "bf16_c128_1x3x46": B.with_(n=1, h=3, w=46, c_half=128, blocks=1),
    "bf16_c128_1x3x47": B.with_(n=1, h=3, w=47, c_half=128, blocks=1),
    "bf16_c256_3x7x7": B.with_(n=3, h=7, w=7, c_half=256, blocks=1),
    "bf16_c512_2x3x5": B.with_(n=2, h=3, w=5, c_half=512, blocks=1),
    # more than 256 tiles of 64 x 64
    "bf16_c128_9x30x31": B.with_(n=9, h=30, w=31, c_half=128, blocks=1),
    # wider than any patch: the im2col kernel
    "bf16_c32_1x2x300": B.with_(n=1, h=2, w=300, blocks=1),
    # 1x1 convs without a kernel of their own
    "bf16_bottleneck_c64_16_3x9x11": NECK.with_(n=3, h=9, w=11, c_half=64, c_mid=16, blocks=1),
    "bf16_bottleneck_c256_64_2x7x7": NECK.with_(n=2, h=7, w=7, c_half=256, c_mid=64, blocks=1),
    # weight gradients: wide images, on flattened pixels and (64 and more) not; the
    # other channel blocks of the 1x1 convs
    "bf16_c64_1x3x63": B.with_(n=1, h=3, w=63, c_half=64, blocks=1),
    "bf16_c64_1x3x64": B.with_(n=1, h=3, w=64, c_half=64, blocks=1),
    "bf16_c32_1x3x79": B.with_(n=1, h=3, w=79, blocks=1),
    "bf16_c32_1x3x80": B.with_(n=1, h=3, w=80, blocks=1),
    "bf16_bottleneck_c64_32_2x7x9": NECK.with_(n=2, h=7, w=9, c_half=64, c_mid=32, blocks=1),
    "bf16_bottleneck_c32_16_2x7x9": NECK.with_(n=2, h=7, w=9, c_half=32, c_mid=16, blocks=2),
    "bf16_bottleneck_c16_16_2x7x9": NECK.with_(n=2, h=7, w=9, c_half=16, c_mid=16, blocks=1),
    "fp32_bottleneck_c32_32_2x7x9": NECK.with_(n=2, h=7, w=9, c_half=32, c_mid=32, blocks=2,
                                               dtype="fp32"),
    "fp32_c64_1x3x56": F.with_(n=1, h=3, w=56, c_half=64, blocks=1),
    "fp32_c64_1x3x62": F.with_(n=1, h=3, w=62, c_half=64, blocks=1),
    "fp32_c16_5x5x13": F.with_(n=5, h=5, w=13, blocks=1),
    "fp32_c32_1x13x5": F.with_(n=1, h=13, w=5, c_half=32, blocks=1),
    "fp32_c64_2x9x21": F.with_(n=2, h=9, w=21, c_half=64, blocks=1),
    "fp32_c128_1x4x19": F.with_(n=1, h=4, w=19, c_half=128, blocks=1),
    "fp32_c128_1x4x20": F.with_(n=1, h=4, w=20, c_half=128, blocks=1),
    "fp32_bottleneck_c64_16_3x9x11": NECK.with_(n=3, h=9, w=11, c_half=64, c_mid=16, blocks=1,
                                                dtype="fp32"),
}


# weight gradients: the widest image whose patch a 3x3 plan takes (registers for its rows;
# fp32, 64 channels: LDS), by type and channel block
WIDEST = {("bf16", 16): 63, ("bf16", 32): 63, ("bf16", 64): 63,
          ("fp32", 16): 95, ("fp32", 32): 63, ("fp32", 64): 61}


def wgrad_kernels(wl):
    """Names of the weight-gradient kernels of one backward."""
    import torch
    from paper_2406_02052_amd import _lib as L

    st = gpu_stage(wl, synth.stage_params(wl, "random"))
    y, d, x, dx = ([st.act().normal_() for _ in range(2)] for _ in range(4))
    L.petra_stage_profile(st.handle, True)
    st.reconstruct_backward(*y, *d, *x, *dx)
    torch.cuda.synchronize()
    return [k[0] for k in L.petra_stage_profile_kernel(st.handle) if k[1] == 2]


@pytest.mark.parametrize("dtype,c,wide", [(*k, d) for k in WIDEST for d in (0, 1)])
def test_widest_weight_gradient(dtype, c, wide):
    base = F if dtype == "fp32" else B
    wl = base.with_(n=1, h=3, w=WIDEST[dtype, c] + wide, c_half=c, blocks=1)
    print(f"case {wl}", flush=True)
    names = wgrad_kernels(wl)
    print(names, flush=True)
    assert all(("wgrad_flat" in k) == (wide == 0) for k in names) and names
    for mode in ("isoF", "isoG") if dtype == "bf16" else ("full",):
        got, want, exact = run_step_parity(wl, bn_affine="random", mode=mode, anchor=False)
        print(check(wl, mode, got, want, exact), flush=True)


@pytest.mark.parametrize("name,mode", [(n, m) for n, wl in CASES.items()
                                       for m in (("isoF", "isoG") if wl.dtype == "bf16" else ("full",))])
def test_stage_step_parity_flat(name, mode):
    wl = CASES[name]
    print(f"case {name} {mode}: {wl}", flush=True)
    got, want, exact = run_step_parity(wl, bn_affine="random", mode=mode, anchor=False)
    print(check(wl, mode, got, want, exact), flush=True)
