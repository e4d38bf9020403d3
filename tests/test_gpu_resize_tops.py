"""The in-place resize with the different numbers of chunks that are computed side by side into scratch (64 to 256), at the edges
of the rule: every tensor changes its size at every step, probed and not, in both directions, against the oracle.  The order
of chunks itself is replayed on the CPU (test_resize_top.py, test_resize_schedule.py)."""
import pytest

from _gpu_harness import Pair
from test_gpu_parity import FP16, FP32, custom

pytestmark = pytest.mark.gpu
CHUNK = 4096

# (chunks computed side by side, tensor sizes)
SETS = {
    "128 of 129": [129 * CHUNK, 128 * CHUNK + 1, 5, CHUNK],
    "128 of 255": [255 * CHUNK - 3, 127 * CHUNK, 128 * CHUNK],
    "256 of 257": [257 * CHUNK - 1, 256 * CHUNK, 255 * CHUNK + 9],
    "256 of 601": [601 * CHUNK - 5, 300 * CHUNK + 2, 1000],
    "256 of 1024": [1024 * CHUNK, 1023 * CHUNK + 1],
    "64, many": [150 * CHUNK] + [70 * CHUNK + 7] * 3 + [333] * 40,
}


@pytest.mark.parametrize("momentum", [0.9, 0.0])
@pytest.mark.parametrize("which", SETS)
def test_parity_when_every_tensor_changes_its_size(which, momentum):
    sizes = SETS[which]
    wl = custom(sizes, name="large_streaming", beta_var=0.0, tau_low=1e-4, tau_high=1e-2, tau_curv=1e30, momentum=momentum)
    p = Pair(wl)
    none = [None] * wl.n_tensors
    for t, scale in enumerate((30.0, 0.03, 30.0, 0.3, 30.0, 0.03), start=1):
        g, z, hz = p.inputs(t)
        p.step([x * scale for x in g], z if t % 2 else none, hz if t % 2 else none, label=f"scale {scale}")
    assert all({row[l] for row in p.code_hist} >= {FP16, FP32} for l in range(len(sizes)))
    p.close()
