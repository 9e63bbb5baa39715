"""A stage step gives the bits of its forward, backward and update called one after
another, on both sides of the rule that chooses one stream or two for it: the largest
half tensor that takes one stream and the next, the widest convs and the next, a second
block, a bottleneck."""
import numpy as np
import pytest

import synth
from tests.test_gpu_stage import _io, gpu_stage

pytestmark = pytest.mark.gpu

B, F = synth.CIFAR_STAGE, synth.BLOCK_FP32
CASES = {
    "bf16_c32_32x16x16": B.with_(n=32, h=16, w=16, blocks=1),
    "bf16_c32_33x16x16": B.with_(n=33, h=16, w=16, blocks=1),
    "bf16_c64_3x8x8": B.with_(n=3, h=8, w=8, c_half=64, blocks=1),
    "bf16_c32_3x8x8_2": B.with_(n=3, h=8, w=8, blocks=2),
    "fp32_c16_8x8x8": F,
    "bf16_neck_3x14x14": synth.IMAGENET_BOTTLENECK_STAGE.with_(n=3, h=14, w=14, blocks=1),
    "fp32_neck_c32_3x14x14": synth.IMAGENET_BOTTLENECK_STAGE.with_(n=3, h=14, w=14, blocks=1,
                                                                   dtype="fp32"),
    "fp32_neck_c64_3x14x14": synth.IMAGENET_BOTTLENECK_STAGE.with_(n=3, h=14, w=14, blocks=1,
                                                                   c_mid=64, dtype="fp32"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_step_equals_separate_calls_bitwise(name):
    import torch
    from paper_2406_02052_amd import to_host

    wl = CASES[name]
    print(f"case {name}: {wl}", flush=True)
    params = synth.stage_params(wl, "random")
    outs = []
    for step in (False, True):
        st = gpu_stage(wl, params)
        x1, x2, _, _ = _io(st, wl, 1)
        yb1, yb2, db1, db2 = _io(st, wl, 2)
        y1, y2, xb1, xb2, dxb1, dxb2 = (st.act() for _ in range(6))
        for _ in range(3):
            if step:
                st.step(x1, x2, y1, y2, yb1, yb2, db1, db2, xb1, xb2, dxb1, dxb2)
            else:
                st.forward(x1, x2, y1, y2)
                st.reconstruct_backward(yb1, yb2, db1, db2, xb1, xb2, dxb1, dxb2)
                st.update()
        torch.cuda.synchronize()
        outs.append([to_host(t) for t in (y1, y2, xb1, xb2, dxb1, dxb2, st.params, st.mom,
                                          st.run_mean, st.run_var)])
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
