"""Thresholds settled inside the update's launch (sets bound by their launches), against the oracle: small tensors read
whole, listed keys of larger ones in registers, more of them than fit, and selections that need histograms; curvature
with ties, zeros, one value, many octaves and denormals."""
import numpy as np
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import FP32, custom

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 5, 63, 64, 65, 257, 1025, 4093, 4095, 4096, 4097, 5000, 8189, 8191, 8192, 8193, 20001, 131073]
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
def test_small_tensors_and_first_steps(pattern, keep):
    wl = custom(SIZES, steps=4, tau_low=0.0, tau_high=0.0, tau_curv=1e30, **keep)
    p = Pair(wl)
    gen = torch.Generator().manual_seed(len(pattern))
    for t in (1, 2, 3, 4):
        g, z, hz = p.inputs(t)
        if t != 3:
            hz = [curvature(pattern, n, gen) for n in SIZES]
            z = [torch.ones(n) for n in SIZES]
        p.step(g, z, hz, label=f"{pattern} {keep}")
    p.close()


def test_more_listed_keys_than_registers_hold():
    """A threshold that jitters widens the predicted band: its lists outgrow the 4096 keys of a workgroup's registers."""
    sizes = [300007, 9000, 1200011, 40]
    wl = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.0)
    p = Pair(wl)
    held = 0
    rng = np.random.default_rng(3)
    for t in range(1, 25):
        g, z, hz = p.inputs(t)
        s = float(1.0 + 0.04 * rng.standard_normal())
        p.step(g, z, [h * s for h in hz], label=f"t={t}")
        held += sum(1 for x in p.gpu.layer_state() if x.sel_outcome == 1 and x.sel_listed > 4096)
    assert held >= 3  # such steps were made, and compared
    p.close()
