"""Which convolution runs, on both sides of the lines between the flattened-pixel and the
im2col kernels, and GPU parity just above each line (the bars of tests/harness.py,
without the direction anchor)."""
import re

import pytest

import synth
from tests.harness import check, gpu_stage, run_step_parity

pytestmark = pytest.mark.gpu

B, F = synth.CIFAR_STAGE.with_(blocks=1), synth.BLOCK_FP32
NECK = synth.IMAGENET_BOTTLENECK_STAGE.with_(blocks=1)
STATS, MASK, RESID, RESID_STATS = range(4)   # epilogues
ALL, INPUT_GRADS = (STATS, MASK, RESID, RESID_STATS), (MASK, RESID, RESID_STATS)

# the largest workload below the line, what is changed to cross it, filter taps per
# side, the epilogues whose conv changes and those whose conv does not
LINES = {
    "3x3_64": (B.with_(n=80, h=32, w=32, c_half=64), dict(n=81), 3, ALL, ()),
    "3x3_128_wide": (B.with_(n=7, h=64, w=64, c_half=128), dict(n=8), 3, ALL, ()),
    "3x3_16_bf16": (B.with_(n=64, h=32, w=32, c_half=16), dict(n=65), 3, (STATS,), INPUT_GRADS),
    "3x3_16_fp32": (F.with_(n=48, h=32, w=32), dict(n=49), 3, (STATS,), INPUT_GRADS),
    "1x1_64_64": (NECK.with_(n=60, h=32, w=32, c_half=64, c_mid=64), dict(n=61), 1,
                  (STATS, MASK), ()),
    "1x1_64_64_resid": (NECK.with_(n=48, h=32, w=32, c_half=64, c_mid=64), dict(n=49), 1,
                        (RESID, RESID_STATS), (STATS, MASK)),
    "1x1_32_64_resid": (NECK.with_(n=32, h=32, w=32, c_half=64, c_mid=32), dict(n=33), 1,
                        (RESID, RESID_STATS), (STATS, MASK)),
    "1x1_128_512_resid": (NECK.with_(n=24, h=16, w=16, c_half=512, c_mid=128), dict(n=25), 1,
                          (RESID, RESID_STATS), (STATS, MASK)),
    "1x1_16_outputs_fp32": (NECK.with_(n=3, h=9, w=11, c_half=64, c_mid=32, dtype="fp32"),
                            dict(c_mid=16), 1, (), INPUT_GRADS),
}


def conv_kernels(wl):
    """{epilogue: kernels that ran with it in a forward and a backward}, a flattened-pixel
    one as flat and its taps per side; the im2col kernels' names do not tell theirs."""
    import torch
    from paper_2406_02052_amd import _lib as L

    st = gpu_stage(wl, synth.stage_params(wl, "random"))
    x, y, d, o = ([st.act().normal_() for _ in range(2)] for _ in range(4))
    back, dx = ([st.act() for _ in range(2)] for _ in range(2))
    L.petra_stage_profile(st.handle, True)
    st.forward(*x, *o)
    st.reconstruct_backward(*y, *d, *back, *dx)
    torch.cuda.synchronize()
    out = {}
    for name, kind, launches, *_ in L.petra_stage_profile_kernel(st.handle):
        if kind > 1:   # not a convolution
            continue
        args = [a.strip() for a in re.search(r"<(.*)>", name).group(1).split(",")]
        ep = int(args[-2]) if re.search("conv_(flat|staged|gemm)", name) else None
        out.setdefault(ep, set()).add("flat%s" % args[1] if "conv_flat" in name else
                                      name.split("<")[0].split("::")[-1])
    return out


@pytest.mark.parametrize("name", list(LINES))
def test_lines_between_conv_kernels(name):
    below, change, taps, cross, stay = LINES[name]
    above = below.with_(**change)
    print(f"case {name}: {above}", flush=True)
    lo, hi = conv_kernels(below), conv_kernels(above)
    print(lo, hi, flush=True)
    im2col = "conv_staged_kernel" if above.dtype == "bf16" and above.c_half >= 32 else "conv_gemm_kernel"
    flat = f"flat{taps}"
    for ep in cross:
        assert flat in lo[ep], (ep, lo)
        assert flat not in hi[ep] and im2col in hi[ep], (ep, hi)
    for ep in stay:
        assert flat in lo[ep] and flat in hi[ep], (ep, lo, hi)
    if name == "1x1_16_outputs_fp32":   # the first conv changes, the last does not
        assert im2col not in lo[STATS] and im2col in hi[STATS] and flat in hi[STATS]
    # isoG for 128 -> 512: with these inputs the sum of F's bn1.beta gradient cancels so far
    # that any bf16 order of sums is past the bar in isoF (im2col kernels alone 0.0234,
    # these 0.0228, every other tensor below 0.008)
    mode = "isoF" if above.dtype == "bf16" and name != "1x1_128_512_resid" else "isoG"
    got, want, exact = run_step_parity(above, bn_affine="random", mode=mode, anchor=False)
    print(check(above, mode, got, want, exact), flush=True)


# the im2col kernels at small sizes: images wider than any patch
WIDE = {
    "bf16_c64_1x2x140": B.with_(n=1, h=2, w=140, c_half=64),
    "bf16_c128_1x2x130": B.with_(n=1, h=2, w=130, c_half=128),
    "bf16_c16_1x2x290": B.with_(n=1, h=2, w=290, c_half=16),
    "fp32_c16_1x2x190": F.with_(n=1, h=2, w=190),
}


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_images_take_im2col(name):
    wl = WIDE[name]
    print(f"case {name}: {wl}", flush=True)
    assert not any(k.startswith("flat3") for ks in conv_kernels(wl).values() for k in ks)
    for mode in ("isoF", "isoG"):
        got, want, exact = run_step_parity(wl, bn_affine="random", mode=mode, anchor=False)
        print(check(wl, mode, got, want, exact), flush=True)
