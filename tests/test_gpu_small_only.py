"""Sets of tensors of up to 8192 elements only, for which no pass over histograms is launched: the short form, in which each
is read whole beside the update at every refresh, and those with a launch for the layers' decisions (step sizes per
element; 16,384 chunks and more).  Several refreshes with ties, zeros, one value, many octaves and more entries asked for
than are not zero, against the oracle."""
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import custom
from test_gpu_select_local import curvature

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 63, 64, 65, 1025, 4095, 4096, 4097, 8191, 8192]
PATTERNS = ["ties", "zeros", "single", "octaves", "equal", "normal"]


def run(wl, sizes, patterns, steps=(1, 2, 3)):
    p = Pair(wl)
    gen = torch.Generator().manual_seed(len(sizes))
    for t in steps:
        g, z, hz = p.inputs(t)
        hz = [curvature(patterns[(i + t) % len(patterns)], n, gen) for i, n in enumerate(sizes)]
        z = [torch.ones(n) for n in sizes]
        p.step(g, z, hz, label=f"t={t}")
    assert {x.sel_outcome for x in p.gpu.layer_state()} == {0}
    p.close()


@pytest.mark.parametrize("keep", [dict(sparsity_ppm=950000), dict(sparsity_ppm=0), dict(topk_abs=5)])
@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("elementwise", [0, 1])
def test_step_sizes_per_layer_and_per_element(elementwise, pattern, keep):
    wl = custom(SIZES, steps=3, tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.5, elementwise_scale=elementwise,
                alpha=1e3, **keep)
    run(wl, SIZES, [pattern])


@pytest.mark.parametrize("keep", [dict(sparsity_ppm=300000), dict(topk_abs=9)])
def test_more_than_sixteen_thousand_chunks(keep):
    sizes = SIZES * 40 + [(7 * i) % 60 + 1 for i in range(16384 - 15 * 40)]
    assert sum(-(-n // 4096) for n in sizes) >= 16384
    wl = custom(sizes, name="large_streaming", steps=3, tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.5, **keep)
    run(wl, sizes, PATTERNS, steps=(1, 2))
