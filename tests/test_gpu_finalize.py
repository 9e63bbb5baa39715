"""GPU parity of the BN finalizes at the edges of their tile counts: stages of 8 x 8
images of 16 channels, whose convs write a partial row per image,
with as many images as one wave, one, two and four tiles per thread of four waves and
a second pass take, and one more of each (bars of tests/harness.py)."""
import pytest

import synth
from tests.harness import check, run_step_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 512, 513, 1024, 1025])
def test_finalize_matches_oracle(n):
    wl = synth.BLOCK_FP32.with_(n=n, h=8, w=8, c_half=16, blocks=1)
    print(f"case {wl}", flush=True)
    got, want, exact = run_step_parity(wl, bn_affine="random", mode="isoF", anchor=False)
    print(check(wl, "isoF", got, want, exact), flush=True)
