"""Sets bound by their launches whose last refresh needed the launch after the update: the next one leaves every threshold
to that launch, small tensors listed whole again.  Refreshes of both kinds in any order, with skipped steps, steps
without a probe and steps that probe only some tensors between them, against the oracle."""
import random

import pytest

from _gpu_harness import Pair
from test_gpu_parity import custom

pytestmark = pytest.mark.gpu

SIZES = [300007, 9000, 40, 70001, 1, 3, 4095, 4096, 4097, 8191, 8192]
HELD = 4096  # listed keys that the update's launch can settle
WAYS = ["calm"] * 6 + ["nudge"] * 3 + ["none", "skip", "small only", "large only"]


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("source", ["hutchinson", "fisher"])
@pytest.mark.parametrize("seed", [1, 2])
def test_refreshes_of_both_kinds_in_turn(seed, source, graph):
    fisher = source == "fisher"
    wl = custom(SIZES, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.0, curvature_source=int(fisher))
    p = Pair(wl, graph=graph)
    rng = random.Random(seed)
    ways = ["calm"] * 4 + [rng.choice(WAYS) for _ in range(30)] + ["jump", "jitter", "jump", "calm", "calm"]
    late, steps, level = False, {False: 0, True: 0}, 1.0
    for t, way in enumerate(ways, start=1):
        # one set of inputs: thresholds stay where they are, to 48 keys, until they are moved out of their bands
        g, z, hz = p.inputs(1, probe=not fisher and way != "none")
        if way == "nudge":
            level *= 1.002
        factor = level * {"jump": 60.0 if t % 2 else 0.02, "jitter": 1.1}.get(way, 1.0)
        if fisher:
            g = [x * factor for x in g]
        elif way != "none":
            hz = [x * factor for x in hz]
            for i, n in enumerate(SIZES):
                if way == "small only" and n > 8192 or way == "large only" and n <= 8192:
                    z[i] = hz[i] = None
        if way == "skip":
            g[3][17] = float("inf")
        res = p.step(g, z, hz, label=f"{way} late={late}", update_curvature=way != "none")
        assert res["skipped"] == int(way == "skip")
        if res["skipped"] or way == "none":
            continue
        steps[late] += 1
        state = [x for x, n in zip(p.gpu.layer_state(), SIZES) if n > 8192 and not (way == "small only" and not fisher)]
        late = any(x.sel_outcome != 1 or x.sel_listed > HELD for x in state)
    assert min(steps.values()) >= 6, steps
    p.close()
