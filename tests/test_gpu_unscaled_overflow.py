"""Gradients that are finite as stored and overflow fp32 when they are unscaled (a loss scale below one): the step
is not skipped, the tensor's variance is not finite, and its precision is therefore FP32.  Tensors of one chunk, of
a few and of many, on either side of the rule that lets the update take the layers' decisions, against the oracle."""
import math

import numpy as np
import pytest

from _gpu_harness import STAT_RTOL, Pair, bits_equal, same_or_both_nan
from _runner import to_numpy
from test_gpu_parity import BF16, FP16, FP32, custom

pytestmark = pytest.mark.gpu

LARGEST = {"local": 1000 * 4096 + 1, "general": 1100 * 4096 - 3}
HEALTHY = (0, 4)  # tensors without an overflow


def compare(p, where):
    for l, (o, g) in enumerate(zip(p.orc.tensors, p.gpu.layer_state())):
        w = (where, l, o.numel)
        assert (g.code, g.prev_code, g.found_inf) == (o.code, o.prev_code, 0), w
        for name, gv, ov in (("var", g.var, float(o.var)), ("v", g.v, float(o.v)), ("mean", g.mean, float(o.mean))):
            assert math.isfinite(gv) == math.isfinite(ov), (w, name, gv, ov)
        if math.isfinite(o.var):
            assert abs(g.var - float(o.var)) <= STAT_RTOL * float(o.var), w
        assert bits_equal(p.gpu.mask[l].cpu().numpy().view(np.uint32), o.mask), w
        assert bits_equal(p.gpu.curv[l].cpu().numpy(), o.curv), w
        assert same_or_both_nan(p.gpu.mom[l].cpu().numpy(), o.mom), w
        gp, op = to_numpy(p.gpu.param(l, g.code)), o.param_view()
        assert same_or_both_nan(gp, op) if o.code == FP32 else bits_equal(gp, op), w


@pytest.mark.parametrize("grad_dtype", [FP32, BF16])
@pytest.mark.parametrize("place", ["first", "chunk0", "last"])
@pytest.mark.parametrize("side", sorted(LARGEST))
def test_variance_of_an_overflowing_gradient_is_not_finite(side, place, grad_dtype):
    sizes = [700, 1000, 4096, 8000, 9000, 4096 * 130 + 5, LARGEST[side]]
    # thresholds far above the variance of the generated gradients (below 1e-2)
    wl = custom(sizes, name="large_streaming", grad_dtype=grad_dtype, tau_low=1.0, tau_high=10.0, tau_curv=1e30,
                loss_scale=0.5)
    p = Pair(wl)
    for t in (1, 2, 3):
        g, z, hz = p.inputs(t)
        if t == 2:
            for l, x in enumerate(g):
                if l not in HEALTHY:
                    x.view(-1)[{"first": 0, "chunk0": 517, "last": x.numel() - 1}[place]] = 2e38
        r = p.step(g, z, hz, check=False, margin_check=False)
        assert not r["skipped"]
        compare(p, (side, place, t))
    # ordinary gradients took every tensor to FP16; the overflow took its tensors to FP32, and their average keeps them there
    assert p.code_hist[0] == [FP16] * len(sizes)
    want = [FP16 if l in HEALTHY else FP32 for l in range(len(sizes))]
    assert p.code_hist[1] == want and p.code_hist[2] == want
    p.close()
