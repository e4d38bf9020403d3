"""Sets on either side of the rule that lets the update take the layers' decisions itself (largest tensor of
1024 chunks / one chunk more), against the oracle: fallback selection, a jump of the curvature, steps without
a probe and with a probe for some tensors only, a skipped step and storage sizes that change."""
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import FP16, FP32, custom

pytestmark = pytest.mark.gpu

LARGEST = {"local": 1024 * 4096 - 5, "general": 1024 * 4096 + 1}


@pytest.mark.parametrize("momentum", [0.9, 0.0])
@pytest.mark.parametrize("side", sorted(LARGEST))
def test_decisions_in_the_update_and_in_the_per_layer_kernel(side, momentum):
    sizes = [5000, 300007, LARGEST[side], 33, 129 * 4096 + 1, 4096]
    wl = custom(sizes, name="large_streaming", beta_var=0.0, tau_low=1e-4, tau_high=1e-2, tau_curv=1e30, momentum=momentum,
                param_dtypes=[FP32, FP16, FP32, FP32, FP16, FP32])
    p = Pair(wl)
    # gradient scale (it decides the codes), factor on Hz, tensors with a probe
    every = [True] * len(sizes)
    plan = [(3.0, 1.0, every), (3.0, 1.0, every), (0.3, 1.0, every), (30.0, 40.0, every), (30.0, 1.0, [False] * len(sizes)),
            (0.3, 1e-3, [True, False, True, True, False, True]), (3.0, 1.0, every)]
    for t, (scale, jump, probed) in enumerate(plan, start=1):
        g, z, hz = p.inputs(t)
        g = [x * scale for x in g]
        if t == 5:  # a skipped step among them
            bad = [x.clone() for x in g]
            bad[2][4096 * 77 + 3] = float("inf")
            p.step(bad, z, hz, label="skipped")
        p.step(g, [a if on else None for a, on in zip(z, probed)], [a * jump if on else None for a, on in zip(hz, probed)],
               label=f"{side} t={t}")
    assert len({row[2] for row in p.code_hist}) == 3
    p.close()


def test_no_applied_step_before_a_skipped_one_and_many_small_tensors():
    # one tensor per workgroup, more tensors than one wave of workgroups, the first call skipped
    wl = custom([1 + 37 * i % 4099 for i in range(700)], name="large_streaming")
    p = Pair(wl)
    g, z, hz = p.inputs(1)
    bad = [x.clone() for x in g]
    bad[699][0] = float("nan")
    p.step(bad, z, hz, label="skipped")
    for t in (2, 3):
        g, z, hz = p.inputs(t)
        none = [None] * wl.n_tensors
        p.step(g, z if t == 2 else none, hz if t == 2 else none)
    p.close()
