"""Thresholds settled inside the update's launch (sets bound by their launches), against the oracle: small tensors read
whole, listed keys of larger ones in registers, more of them than fit, and selections that need histograms; curvature
with ties, zeros, one value, many octaves and denormals."""
import numpy as np
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import FP32, custom

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 5, 63, 64, 65, 257, 1025, 4093, 4095, 4096, 4097, 5000, 8189, 8191, 8192, 8193, 20001]
LARGEST = [131073, 131072]  # chunks: 33 and 32
PATTERNS = ["ties", "zeros", "single", "octaves", "denormal", "equal", "normal"]


def curvature(pattern, n, gen):
    x = torch.randn(n, generator=gen)
    if pattern == "ties":
        return torch.randint(1, 5, (n,), generator=gen).float()
    if pattern == "zeros":
        return x * (torch.rand(n, generator=gen) < 0.1)
    if pattern == "single":
        y = torch.zeros(n)
        y[int(torch.randint(0, n, (1,), generator=gen))] = 3.0
        return y
    if pattern == "octaves":  # far beyond the two octaves of the first window
        return x * torch.exp2(torch.randint(-60, 60, (n,), generator=gen).float())
    if pattern == "denormal":
        return x * 1e-42
    if pattern == "equal":
        return torch.full((n,), -0.5)
    return x


@pytest.mark.parametrize("keep", [dict(sparsity_ppm=950000), dict(sparsity_ppm=300000), dict(sparsity_ppm=0), dict(topk_abs=5)])
@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("largest", LARGEST)
def test_small_tensors_and_first_steps(largest, pattern, keep):
    sizes = SIZES + [largest]
    wl = custom(sizes, steps=4, tau_low=0.0, tau_high=0.0, tau_curv=1e30, **keep)
    p = Pair(wl)
    gen = torch.Generator().manual_seed(len(pattern))
    for t in (1, 2, 3, 4):
        g, z, hz = p.inputs(t)
        if t != 3:
            hz = [curvature(pattern, n, gen) for n in sizes]
            z = [torch.ones(n) for n in sizes]
        p.step(g, z, hz, label=f"{pattern} {keep}")
    p.close()


@pytest.mark.parametrize("sizes", [[300007, 9000, 1200011, 40], [131072, 9000, 131071, 40]])
def test_more_listed_keys_than_registers_hold(sizes):
    """A threshold that jitters widens the predicted band: its lists outgrow the 4096 keys of a workgroup's registers."""
    wl = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.0)
    p = Pair(wl)
    held = 0
    rng = np.random.default_rng(3)
    for t in range(1, 25):
        g, z, hz = p.inputs(t)
        s = float(1.0 + 0.06 * rng.standard_normal())
        p.step(g, z, [h * s for h in hz], label=f"t={t}")
        held += sum(1 for x in p.gpu.layer_state() if x.sel_outcome == 1 and x.sel_listed > 4096)
    assert held >= 3  # such steps were made, and compared
    p.close()


def test_histograms_at_every_step():
    """Curvature that jumps by a factor of 4000 and back: predictions fail, the selection counts, lists and refines."""
    sizes = [131072, 100352, 8193, 20000, 500]
    wl = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.0)
    p = Pair(wl)
    fell_back = 0
    for t in range(1, 13):
        g, z, hz = p.inputs(t)
        if t % 4 == 0:
            hz = [h * 0 if i == 1 else h for i, h in enumerate(hz)]  # fewer non-zero keys than are to be kept
        p.step(g, z, [h * (40.0 if t % 2 else 0.01) for h in hz], label=f"t={t}")
        fell_back += sum(1 for x in p.gpu.layer_state() if x.sel_outcome in (2, 3, 4, 6))
    assert fell_back >= 30
    p.close()
