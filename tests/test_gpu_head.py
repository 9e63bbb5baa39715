"""GPU parity of the loss head at the edges of its thread groups: image counts that no
group of images divides, the smallest and largest class counts, one pixel per channel.
Held: the losses, and the momentum (after one backward: the gradient) of the head's
parameters and of the BN gain that its input gradient reaches first, at the fp32 bar.
(Not the increments: that gain's are some 2e-4 on a value of 1, whose last fp32 bit is
3e-4 of them.)"""
import pytest

import synth
from tests.harness import TOL, rel
from tests.test_gpu_net import affine_params, run_both

pytestmark = pytest.mark.gpu

BASE = synth.REVNET18_SCHEDULE.with_(dtype="fp32", blocks_per_stage=1, lr=0.02)


@pytest.mark.parametrize("n,h,widths,classes", [(9, 16, (16, 32), 2), (17, 8, (16, 32), 64),
                                                (67, 2, (16, 32), 33), (5, 8, (128,), 10)])
def test_head_matches_oracle(n, h, widths, classes):
    wl = BASE.with_(n=n, h=h, w=h, widths=widths, classes=classes)
    print(f"case {wl}", flush=True)
    names, params = affine_params(wl)
    J = len(widths)
    ref, oloss, net, gloss = run_both(wl, names, params, 1, 2 * J - 1)
    want = {nm: b for st in ref.stages for nm, b in zip(st.names, st.buf)}
    got = dict(zip(names, net.get_momentum()))
    for a, b in zip(gloss, oloss):
        assert (a is None) == (b is None)
        assert b is None or abs(a - b) <= TOL["fp32"] * abs(b), (a, b)
    for nm in (f"s{J - 1}.fc.weight", f"s{J - 1}.fc.bias", f"s{J - 1}.b0.G.bn1.gamma"):
        e = rel(got[nm], want[nm])
        print(nm, e, flush=True)
        assert e <= TOL["fp32"], (nm, e)
