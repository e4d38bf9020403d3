"""Power iteration on more tensors than travel as kernel arguments: the pinned copy (several calls in flight, each
with other vectors), the arguments while a stream is captured, and the cost of a call with thousands of tensors."""
import time

import pytest
import torch

import paper_2508_16905_amd as ta
from workloads.configs import _DEFAULT_HYPER

pytestmark = pytest.mark.gpu
K = 2


def vectors(n, numel, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    us = [torch.randn(K, numel, device="cuda", generator=gen) for _ in range(n)]
    hus = [torch.randn(K, numel, device="cuda", generator=gen) for _ in range(n)]
    arr = (ta.PowerTensor * n)()
    for a, u, h in zip(arr, us, hus):
        a.u, a.hu, a.stride = u.data_ptr(), h.data_ptr(), numel
    return us, hus, arr


def make(n, numel, stream=None):
    return ta.TriAccel(dict(_DEFAULT_HYPER, power_k=K), [torch.zeros(numel, device="cuda") for _ in range(n)], stream=stream)


def orthonormal(hus):
    # the basis of ordered Gram-Schmidt in fp64
    out = []
    for h in hus:
        q, r = torch.linalg.qr(h.double().cpu().T)
        out.append((q * torch.sign(torch.diagonal(r))).T)
    return out


def check(us, hus):
    for u, want in zip(us, orthonormal(hus)):
        # fp64 sums, one rounding to fp32, as in tests/test_gpu_power_args.py
        assert torch.allclose(u.cpu().double(), want, rtol=2.0 ** -23, atol=1e-12)


@pytest.mark.parametrize("n", [256, 257, 300])
def test_calls_in_flight_keep_their_own_pointers(n):
    opt = make(n, 44)
    sets = [vectors(n, 44, 100 * n + i) for i in range(10)]  # more than there are staging buffers
    torch.cuda.synchronize()
    for _, _, arr in sets:
        ta.binding.triaccel_power_iter(opt.handle, arr, K, False)
    torch.cuda.synchronize()
    for us, hus, _ in sets:
        check(us, hus)
    opt.close()


@pytest.mark.parametrize("n", [200, 300])
def test_capture_and_replay(n):
    stream = torch.cuda.Stream()
    opt = make(n, 44, stream)
    us, hus, arr = vectors(n, 44, n)
    other_us, other_hus, other = vectors(n, 44, n + 1)
    torch.cuda.synchronize()
    ta.binding.triaccel_power_iter(opt.handle, other, K, False)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        ta.binding.triaccel_power_iter(opt.handle, arr, K, False)
    for replay in range(3):
        for u in us:
            u.normal_()
        for h in hus:
            h.normal_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(us, hus)
        # ordinary calls between the replays, with vectors of their own
        ta.binding.triaccel_power_iter(opt.handle, other, K, False)
        torch.cuda.synchronize()
        check(other_us, other_hus)
    opt.close()


def test_cost_of_thousands_of_tensors():
    def call_us(n):
        opt = make(n, 3000)
        us, hus, arr = vectors(n, 3000, 7)
        run = lambda: ta.binding.triaccel_power_iter(opt.handle, arr, K, False)  # noqa: E731
        times = []
        for _ in range(9):
            run()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(40):
                run()
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t0) / 40 * 1e6)
        opt.close()
        return sorted(times)[4]

    small, large = call_us(1000), call_us(4000)
    # the kernels' work grows by 4; with a launch for every 128 tensors 38 -> 133 us (3.5), with the copy 42 -> 94 (2.2)
    assert large < 2.9 * small, (small, large)
