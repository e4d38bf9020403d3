"""Ends of tensors that are no multiple of four elements: every place in a row, a wavefront and a chunk where the last
one to three elements can lie, against the oracle, and nothing written beside them."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2508_16905_amd as ta
from _gpu_harness import Pair
from test_gpu_parity import BF16, FP16, FP32, custom

pytestmark = pytest.mark.gpu

ENDS = [0, 252, 256, 1020, 1024, 2044, 3068, 3072, 4092, 4096, 8192, 12284]
SIZES = [e + r for e in ENDS for r in (1, 2, 3)] + [4, 1028, 4100]


@pytest.mark.parametrize("form", ["hutchinson", "fisher", "elementwise", "no momentum"])
@pytest.mark.parametrize("store", [FP32, BF16, FP16])
def test_every_place_of_the_end(store, form):
    tau = {FP32: (0.0, 0.0), BF16: (0.0, 1e30), FP16: (1e30, 1e30)}[store]
    wl = custom(SIZES, name="large_streaming", tau_low=tau[0], tau_high=tau[1], tau_curv=1e30, loss_scale=1.0,
                param_dtypes=[store] * len(SIZES), momentum=0.0 if form == "no momentum" else 0.9,
                curvature_source=int(form == "fisher"), elementwise_scale=int(form == "elementwise"))
    p = Pair(wl, grad_dtypes=[(FP32, BF16, FP16)[(i // 3 + i) % 3] for i in range(len(SIZES))])
    for t in (1, 2, 3):
        g, z, hz = p.inputs(t, probe=form != "fisher")
        p.step(g, z, hz, label=form)
    p.close()


GAP = 128  # elements between two tensors of the arenas below


@pytest.mark.parametrize("momentum", [0.9, 0.0])
def test_nothing_is_written_past_the_end(momentum):
    """Storage sizes change at every step (scratch and in-place rewriting of the longest tensor included)."""
    numels = SIZES + [4096 * 200 + 3]
    offs = np.cumsum([0] + [-(-n // 128) * 128 + GAP for n in numels])
    size = int(offs[-1])
    dev = torch.device("cuda:0")
    hyper = dict(custom([1]).hyper, beta_var=0.0, tau_low=0.0, tau_high=1e-4, tau_curv=1e30, momentum=momentum)
    inside = torch.zeros(size, dtype=torch.bool, device=dev)
    for o, n in zip(offs, numels):
        inside[o:o + n] = True
    arena = {k: torch.full((size,), 0x5a5a5a5a, dtype=torch.int32, device=dev) for k in ("param", "mom", "curv")}
    for a in arena.values():
        a[inside] = 0
    mask = torch.full((size // 32,), 0x5a5a5a5a, dtype=torch.int32, device=dev)
    used = inside.view(-1, 32).any(1)
    gen = torch.Generator(device=dev).manual_seed(5)
    z = torch.ones(size, device=dev)
    arr = (ta.Tensor * len(numels))()
    for code in (FP32, BF16, FP32, FP32):
        grad = torch.randn(size, generator=gen, device=dev) * (1e-1 if code == FP32 else 1e-3)
        for t, o, n in zip(arr, offs, numels):
            t.param, t.mom, t.curv = (arena[k].data_ptr() + 4 * int(o) for k in ("param", "mom", "curv"))
            t.grad, t.z, t.hz = (x.data_ptr() + 4 * int(o) for x in (grad, z, grad))
            t.mask = mask.data_ptr() + int(o) // 8
            t.numel, t.grad_dtype, t.param_dtype = n, FP32, FP32
        if code == FP32 and "handle" not in locals():
            handle = ta.triaccel_init(ta.Config.from_hyper(hyper), arr, torch.cuda.current_stream().cuda_stream)
        ta.triaccel_step(handle, arr, 0.1, 1.0, 96, 800, 1000, True)
        torch.cuda.synchronize()
        state = ta.triaccel_layer_state(handle, len(numels))
        assert {x.code for x, n in zip(state, numels) if n > 3} == {code}  # a few elements vary too little
        for k, a in arena.items():
            assert bool((a[~inside] == 0x5a5a5a5a).all()), k
        assert bool((mask[~used] == 0x5a5a5a5a).all())
    ta.triaccel_destroy(handle)


@pytest.mark.parametrize("code", [FP32, BF16, FP16])
def test_conversion_of_every_length(code):
    kind = {FP32: torch.float32, BF16: torch.bfloat16, FP16: torch.float16}[code]
    for n in SIZES:
        src = torch.randn(n, device="cuda:0")
        dst = torch.full((n + GAP,), -7.0, dtype=kind, device="cuda:0")
        ta.triaccel_cast_f32(src.data_ptr(), dst.data_ptr(), n, code, torch.cuda.current_stream().cuda_stream)
        assert torch.equal(dst[:n], src.to(kind)), n
        assert bool((dst[n:] == -7.0).all()), n


@pytest.mark.parametrize("k", [1, 3, 8])
def test_power_iteration_of_every_length(k):
    """Against ordered Gram-Schmidt in 64 bits.  The products are well conditioned (normal entries, n >= 16 k), so both
    routes give the fp64 result to some 1e-14 and the stored value is its rounding, 6e-8 of it, or the next one."""
    numels = [n for n in SIZES if n >= 16 * k]
    gen = torch.Generator(device="cuda:0").manual_seed(k)
    vec = (ta.PowerTensor * len(numels))()
    keep = []
    for v, n in zip(vec, numels):
        stride = -(-n // 4) * 4
        u = torch.randn(k, stride, generator=gen, device="cuda:0")
        hu = torch.randn(k, stride, generator=gen, device="cuda:0")  # the padding must not be read as data
        keep.append((u, hu, u.clone()))
        v.u, v.hu, v.stride = u.data_ptr(), hu.data_ptr(), stride
    info = torch.zeros(len(numels), ctypes.sizeof(ta.PowerInfo) // 4, device="cuda:0")
    ta.triaccel_power_iter_static(vec, numels, k, info.data_ptr(), torch.cuda.current_stream().cuda_stream)
    for (u, hu, before), n in zip(keep, numels):
        q = []
        for j in range(k):
            w = hu[j, :n].double()
            for _ in range(2):
                for p in q:
                    w = w - (p @ w) * p
            q.append(w / w.norm())
        want = torch.stack(q)
        assert float((u[:, :n].double() - want).abs().max() / want.abs().max()) < 2 * 2.0 ** -24 + 1e-11, n
        assert torch.equal(u[:, n:], before[:, n:]), n
