"""Weight gradients of the layers that share a launch: workgroups per launch, and the same
bits however the backward is called (one, two or three streams, graph replay, in place,
inside a step)."""
import re

import numpy as np
import pytest

import synth
from tests.harness import gpu_stage
from tests.test_gpu_stage import _io

pytestmark = pytest.mark.gpu

B, F = synth.CIFAR_STAGE, synth.BLOCK_FP32
NECK = synth.IMAGENET_BOTTLENECK_STAGE


def launches_3x3(wl):
    """[(layers, splits of all of them)] per launch of each flattened-pixel 3x3 kernel in one
    backward, from the operations and the bytes that the profile counts for it: operands,
    and 4 bytes a split and weight."""
    import torch
    from paper_2406_02052_amd import _lib as L

    st = gpu_stage(wl, synth.stage_params(wl, "random"))
    y1, y2, d1, d2 = _io(st, wl, 1)
    out = [st.act() for _ in range(4)]
    L.petra_stage_profile(st.handle, True)
    st.reconstruct_backward(y1, y2, d1, d2, *out)
    torch.cuda.synchronize()
    esz, m = (2 if wl.dtype == "bf16" else 4), wl.n * wl.h * wl.w
    o, r, s, i = max(wl.conv_layers(), key=lambda t: t[1])
    numel = o * r * s * i
    res = []
    for name, _, launches, _, flops, nbytes in L.petra_stage_profile_kernel(st.handle):
        if re.search(r"wgrad_flat.*(bf16_t|float), 3,", name):
            layers = flops / (2.0 * m * numel)
            splits = (nbytes - layers * esz * m * (i + 2 * o)) / (4.0 * numel)
            res.append((round(layers / launches, 3), round(splits / launches, 3)))
    return res


# the 3x3 layers of one launch, and their workgroups per split
SHARED = {
    "bottleneck_one_block": (NECK.with_(n=37, h=23, w=23, blocks=1), 2, 1),
    "two_functions_one_block": (B.with_(n=64, h=28, w=28, c_half=64, blocks=1), 4, 1),
    "function_of_four_blocks": (B.with_(n=64, h=28, w=28, c_half=64, blocks=4), 2, 1),
    "fp32_function_of_four_blocks": (F.with_(n=32, h=32, w=32, c_half=32, blocks=4), 2, 1),
    "small_stage_kept": (B.with_(n=64, h=14, w=14, c_half=128, blocks=1), 4, 4),
}


@pytest.mark.parametrize("name", list(SHARED))
def test_launch_has_a_workgroup_for_every_cu(name):
    wl, layers, per = SHARED[name]
    print(f"case {name}: {wl}", flush=True)
    got = launches_3x3(wl)
    print(got, flush=True)
    assert len(got) == 1 and got[0][0] == layers
    assert 0.9 * 256 <= got[0][1] * per <= 256


MODES = {
    "bf16_c64_3x28x28_b3": B.with_(n=3, h=28, w=28, c_half=64, blocks=3),
    "bf16_c128_5x8x8_b2": B.with_(n=5, h=8, w=8, c_half=128, blocks=2),
    "bf16_c32_9x32x32_b3": B.with_(n=9, h=32, w=32, blocks=3),
    "bf16_c64_9x16x16_b4": B.with_(n=9, h=16, w=16, c_half=64, blocks=4),
    "bf16_c64_2x9x64_b2": B.with_(n=2, h=9, w=64, c_half=64, blocks=2),
    "bf16_neck_3x23x23_b1": NECK.with_(n=3, h=23, w=23, blocks=1),
    "bf16_neck_24x23x23_b3": NECK.with_(n=24, h=23, w=23, blocks=3),
    "bf16_neck_c256_64_2x9x64_b2": NECK.with_(n=2, h=9, w=64, c_half=256, c_mid=64, blocks=2),
    "fp32_c32_20x32x32_b2": F.with_(n=20, h=32, w=32, c_half=32, blocks=2),
    "fp32_c16_8x8x8_b3": F.with_(blocks=3),
}


@pytest.mark.parametrize("name", list(MODES))
def test_stream_modes_bitwise(name):
    import torch
    from paper_2406_02052_amd import to_host

    wl = MODES[name]
    print(f"case {name}: {wl}", flush=True)
    params = synth.stage_params(wl, "random")
    res = []
    for streams, graphs, call in ((1, False, "apart"), (1, False, "in place"), (2, False, "apart"),
                                  (2, False, "in place"), (3, False, "apart"), (3, False, "in place"),
                                  (3, True, "in place"), (1, False, "step"), (2, False, "step")):
        st = gpu_stage(wl, params)
        st.set_streams(streams)
        st.set_graphs(graphs)
        y1, y2, d1, d2 = _io(st, wl, 21)
        a = [t.clone() for t in (y1, y2, d1, d2)]
        out = a if call == "in place" else [st.act() for _ in range(4)]
        f = [t.clone() for t in (y1, y2)] + [st.act(), st.act()]
        for _ in range(2):
            for t, s in zip(a, (y1, y2, d1, d2)):
                t.copy_(s)
            if call == "step":
                st.step(*f, *a, *out)
            else:
                st.reconstruct_backward(*a, *out)
                st.update()
        torch.cuda.synchronize()
        res.append((streams, graphs, call, [to_host(t) for t in out] +
                    [t.cpu().numpy() for t in (st.params, st.mom, st.run_mean, st.run_var)]))
    for mode in res[1:]:
        for a, b in zip(res[0][3], mode[3]):
            assert np.array_equal(a, b), mode[:3]
