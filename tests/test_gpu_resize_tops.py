"""The in-place resize with the different numbers of chunks that are computed side by side into scratch (64 to 256), at the edges
of the rule: every tensor changes its size at every step, probed and not, in both directions, against the oracle; with step sizes per
element too, where the resize is a launch item of another kernel and follows the decisions of k_decide_select.  The order
of chunks itself is replayed on the CPU (test_resize_top.py, test_resize_schedule.py)."""
import pytest

from _gpu_harness import Pair
from test_gpu_parity import FP16, FP32, custom
from test_resize_schedule import lib, plan  # noqa: F401  (lib is the fixture)

pytestmark = pytest.mark.gpu
CHUNK = 4096

# (chunks computed side by side, tensor sizes)
SETS = {
    "128 of 129": (128, [129 * CHUNK, 128 * CHUNK + 1, 5, CHUNK]),
    "128 of 255": (128, [255 * CHUNK - 3, 127 * CHUNK, 128 * CHUNK]),
    "256 of 257": (256, [257 * CHUNK - 1, 256 * CHUNK, 255 * CHUNK + 9]),
    "256 of 601": (256, [601 * CHUNK - 5, 300 * CHUNK + 2, 1000]),
    "256 of 1024": (256, [1024 * CHUNK, 1023 * CHUNK + 1]),
    "64, many": (64, [150 * CHUNK] + [70 * CHUNK + 7] * 3 + [333] * 40),
    # more than 4096 chunks in the set: at most a quarter of the longest tensor
    "128 of 601, long": (128, [601 * CHUNK - 5] * 6 + [600 * CHUNK + 3, 1000]),
}


@pytest.mark.parametrize("which,momentum,elementwise", [(w, m, 0) for w in list(SETS)[:-1] for m in (0.9, 0.0)] + [
    ("128 of 601, long", 0.9, 0), ("128 of 129", 0.0, 1), ("128 of 255", 0.9, 1), ("256 of 601", 0.9, 1), ("64, many", 0.9, 1)])
def test_parity_when_every_tensor_changes_its_size(lib, which, momentum, elementwise):  # noqa: F811
    top, sizes = SETS[which]
    chunks = [-(-n // CHUNK) for n in sizes]
    assert plan(lib, (max(chunks), sum(chunks), len(chunks)))[1] == top
    wl = custom(sizes, name="large_streaming", beta_var=0.0, tau_low=1e-4, tau_high=1e-2, tau_curv=1e30, momentum=momentum,
                elementwise_scale=elementwise)
    p = Pair(wl)
    none = [None] * wl.n_tensors
    scales = (30.0, 0.03, 30.0, 0.3, 30.0, 0.03)
    for t, scale in enumerate(scales[:4] if which.endswith("long") else scales, start=1):
        g, z, hz = p.inputs(t)
        probed = t % 3 != 0 if elementwise else t % 2 != 0
        p.step([x * scale for x in g], z if probed else none, hz if probed else none, label=f"scale {scale}")
    assert all({row[l] for row in p.code_hist} >= {FP16, FP32} for l in range(len(sizes)))
    p.close()
