"""Probed steps of short sets, whose statistics and curvature average are taken in one launch before it is known whether the
step is skipped: curvature, mask and key lists of skipped steps against the oracle, on both sides of the rule (512 pieces of
4096 elements, 256 of a tensor), for all gradient precisions, tensors without a probe, bands and histograms."""
import pytest
import torch

from _gpu_harness import Pair
from test_gpu_parity import custom

pytestmark = pytest.mark.gpu

RAGGED = [1, 3, 31, 33, 127, 129, 1023, 1026, 4095, 4096, 4097, 8191, 8192, 8195, 40961]
CHUNKS = sum(-(-n // 4096) for n in RAGGED)


def sizes_of(chunks):
    if chunks in (256, 257):  # of one tensor
        return RAGGED + [4096 * chunks - 5]
    return RAGGED + ([4096 * 250 - 3, 4096 * (chunks - CHUNKS - 250) - 5] if chunks else [])


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("source", ["hutchinson", "fisher"])
@pytest.mark.parametrize("chunks", [0, 256, 257, 512, 513])
def test_skipped_probed_steps_change_nothing(chunks, source, graph):
    fisher = source == "fisher"
    sizes = sizes_of(chunks)
    dtypes = [(2, 1, 0)[i % 3] for i in range(len(sizes))]
    wl = custom(sizes, name="large_streaming", steps=16, tau_low=0.0, tau_high=0.0, tau_curv=1e30, beta_curv=0.5,
                curvature_source=int(fisher))
    p = Pair(wl, graph=graph, grad_dtypes=dtypes)
    gen = torch.Generator().manual_seed(chunks)
    skips = {1, 3, 8, 9, 12, 15}  # the first call, with thresholds unknown, with bands, twice in a row
    for t in range(1, 17):
        g, z, hz = p.inputs(1 + t % 2, probe=not fisher)
        if not fisher and t in (12, 13):
            for i in range(0, len(sizes), 2):
                z[i] = hz[i] = None
        if t == 14:  # out of its band
            g, hz = ([x * 8 for x in g], hz) if fisher else (g, [x * 60 for x in hz])
        if t in skips:
            i = int(torch.randint(len(sizes), (1,), generator=gen))
            g[i][int(torch.randint(sizes[i], (1,), generator=gen))] = (float("nan"), float("inf"))[t % 2]
        assert p.step(g, z, hz, label=f"t={t}")["skipped"] == int(t in skips)
    p.close()


def test_workspace_on_both_sides_of_the_rule():
    """Old curvature and masks are only put aside, 4.1 bytes per element, in sets that take both in one launch."""
    import paper_2508_16905_amd as ta
    from workloads.configs import _DEFAULT_HYPER

    config = ta.binding.Config.from_hyper(_DEFAULT_HYPER)
    arena = torch.zeros(4 * 512 * 4096, dtype=torch.uint8, device="cuda")  # never read: no step is made

    def used(*chunks):
        table = []
        for c in chunks:
            t = ta.binding.Tensor()
            t.param = t.grad = t.curv = t.mom = t.mask = arena.data_ptr()
            t.numel, t.grad_dtype, t.param_dtype = 4096 * c, ta.FP32, ta.FP32
            table.append(t)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        handle = ta.binding.triaccel_init(config, table)
        got = before - torch.cuda.mem_get_info()[0]
        ta.binding.triaccel_destroy(handle)
        return got

    used(1)
    mib = 1 << 20  # allocations are whole 2 MiB
    # 4.1 MiB (1 MiB = 256 pieces, 4.125 times) less scratch of the resize: 128 chunks of 16 KB a tensor of 256, 256 of 257
    assert used(256) - used(257) > 0
    assert used(256, 256) - used(256, 257) > 2 * mib
    assert used(256, 255, 1) - used(256, 255, 2) > 6 * mib  # more than 512 pieces in all, the same scratch
