"""Pointers of the power iteration as kernel arguments (up to 128 tensors) and through the table (more), and
tensors around the edges of a Gram segment: both entry points against torch in fp64, and against each other
bit for bit."""
import ctypes
import pytest
import torch

import paper_2508_16905_amd as ta
from workloads.configs import _DEFAULT_HYPER

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(127, 2), (128, 5), (129, 5), (255, 3)])
def test_both_ways_of_passing_the_pointers(n, k):
    gen = torch.Generator().manual_seed(n * 10 + k)
    edges = [16383, 16384, 16385, 4095, 4097, 5 * 4096 + 3, 8 * 4096 + 1]
    numel = [edges[i % 7] if i < 14 else 40 + 31 * i for i in range(n)]
    us = [torch.randn(k, (m + 3) // 4 * 4, generator=gen).cuda() for m in numel]
    hus = [torch.randn(k, u.shape[1], generator=gen).cuda() for u in us]
    for m, u, h in zip(numel, us, hus):
        u[:, m:] = float("nan")  # the padding is neither read into a result nor written
        h[:, m:] = float("nan")
    want = []
    for m, h in zip(numel, hus):
        q, r = torch.linalg.qr(h[:, :m].double().T)
        want.append((q * torch.sign(torch.diagonal(r))).T)
    other = [u.clone() for u in us]
    gpu = ta.TriAccel(dict(_DEFAULT_HYPER, power_k=k), [torch.zeros(m, device="cuda") for m in numel])
    gpu.power_iter(us, hus, k)
    info = gpu.power_state()
    gpu.close()
    vec = (ta.PowerTensor * n)()
    for v, u, h in zip(vec, other, hus):
        v.u, v.hu, v.stride = u.data_ptr(), h.data_ptr(), u.shape[1]
    out = torch.zeros(n, ctypes.sizeof(ta.PowerInfo) // 4, device="cuda")
    ta.triaccel_power_iter_static(vec, numel, k, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    out = out.cpu()
    for i, m in enumerate(numel):
        assert torch.equal(us[i][:, :m], other[i][:, :m]), i
        # fp64 sums, one rounding to fp32: half a unit of 2^-24 per element, and the conditioning of random
        # vectors (below 10) squared times 1e-15
        assert torch.allclose(us[i][:, :m].double(), want[i], rtol=2.0 ** -23, atol=1e-12), i
        assert list(out[i, :k]) == [float(info[i].rayleigh[j]) for j in range(k)], i
