"""A configuration whose precision rule always says FP32 (tau_high <= 0) makes no launches for tensors that change their
storage size, once all layers are FP32: layers that start in 16 bits, and a state restored from such a start into a
handle that had left the launches out, also in its captured steps."""
import pytest
import torch

import paper_2508_16905_amd as ta
from _gpu_harness import Pair, bits_equal
from test_gpu_parity import BF16, FP16, FP32, custom

pytestmark = pytest.mark.gpu

SIZES = {"local": [4096 * 200 + 3, 5000, 40, 4096 * 20], "general": [4096 * 1025 + 7, 4096 * 130, 33]}


@pytest.mark.parametrize("form", ["local", "general", "elementwise"])
@pytest.mark.parametrize("start", [FP32, BF16, FP16])
def test_steps_from_every_start(form, start):
    sizes = SIZES["general" if form == "general" else "local"]
    wl = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=0.1, param_dtypes=[start] * len(sizes),
                elementwise_scale=int(form == "elementwise"))
    p = Pair(wl)
    for t in (1, 2, 3):
        g, z, hz = p.inputs(t, probe=t != 2)
        p.step(g, z, hz)
    assert p.code_hist[-1] == [FP32] * len(sizes)
    p.close()


@pytest.mark.parametrize("graph", [False, True])
def test_restored_state_brings_the_launches_back(graph):
    sizes = SIZES["local"]
    low = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, param_dtypes=[BF16] * len(sizes))
    full = custom(sizes, name="large_streaming", tau_low=0.0, tau_high=0.0, tau_curv=1e30, param_dtypes=[FP32] * len(sizes))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        params = [low.init_param(l).cuda() for l in range(len(sizes))]
        a = ta.TriAccel(low.hyper, params, stream=stream)
        b = ta.TriAccel(full.hyper, [full.init_param(l).cuda() for l in range(len(sizes))], stream=stream)
        b.set_graph(graph)
        table = lambda o, t: o.make_table([low.grad(t, l, 1.0).cuda() for l in range(len(sizes))], None, None)  # noqa: E731
        one, two = table(b, 1), table(b, 2)
        args = dict(lr=0.1, loss_scale=1.0, mem_used_bytes=1, mem_total_bytes=2, update_curvature=False)
        for _ in range(3):
            b.step_table(one, **args)  # without the launches; captured if `graph`
        blob = a.get_state()
        torch.cuda.synchronize()
        for i in range(len(sizes)):
            for dst, src in ((b.buf[i], a.buf[i]), (b.curv[i], a.curv[i]), (b.mom[i], a.mom[i]), (b.mask[i], a.mask[i])):
                dst.copy_(src)
        b.set_state(blob)
        same = table(a, 1), table(a, 2)
        for mine, theirs in ((same[0], one), (same[1], two)):
            a.step_table(mine, **args)
            b.step_table(theirs, **args)
        torch.cuda.synchronize()
        assert [x.code for x in b.layer_state()] == [FP32] * len(sizes)
        for i in range(len(sizes)):
            assert bits_equal(a.param(i, FP32).cpu().numpy(), b.param(i, FP32).cpu().numpy()), i
            assert bits_equal(a.mom[i].cpu().numpy(), b.mom[i].cpu().numpy()), i
    a.close()
    b.close()
