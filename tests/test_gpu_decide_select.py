"""Step sizes per element on sets whose layers' decisions and thresholds are taken in one launch before the update: bands,
histograms, fewer entries than are to be kept, skipped steps and steps that probe some tensors only, against the oracle; short
sets (statistics and curvature in one launch, late selections), longer ones, and tensors at the rule's edge (4096 pieces)."""
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import custom

pytestmark = pytest.mark.gpu

SHORT = [300007, 9000, 40, 70001, 1, 3, 4095, 4096, 4097, 8191, 8192]
SETS = {"short": SHORT, "longer": SHORT + [4096 * 1000 + 7], "edge": [4096 * 4096 - 3, 9001, 77], "beyond": [4096 * 4096 + 1, 9001, 77]}
WAYS = ["skip"] + ["calm"] * 4 + ["jump", "calm", "skip", "calm", "calm", "few", "calm", "large only", "small only", "none", "skip", "calm", "jump"]


@pytest.mark.parametrize("which,source,graph", [(w, s, g) for w in ("short", "longer") for s in ("hutchinson", "fisher")
                                                for g in (False, True)] + [("edge", "hutchinson", False), ("beyond", "hutchinson", False)])
def test_steps_of_every_kind(which, source, graph):
    fisher = source == "fisher"
    sizes = SETS[which]
    wl = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.0, curvature_source=int(fisher),
                elementwise_scale=1, alpha=1e2)
    p = Pair(wl, graph=graph)
    ways = WAYS if which in ("short", "longer") else WAYS[:9]
    outcomes = set()
    for t, way in enumerate(ways, start=1):
        g, z, hz = p.inputs(1, probe=not fisher and way != "none")
        if way == "jump":
            g, hz = ([x * 7 for x in g], hz) if fisher else (g, [x * 60 for x in hz])
        if way == "few":  # fewer entries that are not zero than are to be kept
            for x in (g if fisher else hz):
                x[x.numel() // 50:] = 0
        for i, n in enumerate(sizes):
            if not fisher and (way == "small only" and n > 8192 or way == "large only" and n <= 8192):
                z[i] = hz[i] = None
        if way == "skip":
            g[len(g) - 1][0] = float("nan")
        res = p.step(g, z, hz, label=f"{way} t={t}", update_curvature=way != "none")
        assert res["skipped"] == int(way == "skip")
        now = {x.sel_outcome for x, n in zip(p.gpu.layer_state(), sizes) if n > 8192}
        if way == "few":
            assert now == {6}, now
        if way == "jump" and ways[t - 4:t - 1] == ["calm"] * 3:  # out of its band
            assert now == {3}, now
        if t > 1 and ways[t - 2] == "few":  # the band reaches down to the zeros of the step before: too many keys
            assert 5 in now, now
        outcomes |= now
    assert {1, 2} <= outcomes, outcomes
    p.close()


def test_profiled_steps_take_the_same_way():
    wl = custom(SHORT, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.5, elementwise_scale=1)
    p = Pair(wl)
    for t in range(1, 7):
        p.gpu.set_profiling(t % 2)  # an event at every boundary: statistics and curvature are two launches again
        g, z, hz = p.inputs(1 + t % 2)
        if t in (3, 4):
            g[0][5] = float("inf")
        p.step(g, z, hz, label=f"t={t}")
    torch.cuda.synchronize()
    p.close()
