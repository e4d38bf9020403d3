"""The power iteration without a handle and with one, bit for bit, whatever number of vectors the handle is sized for.
The products of a layer are nearly the same vector (pivots of some 1e-8 of the squared norms), so that sums that were
added in another order show: their rounding errors come out some 1e8 times larger in the factors."""
import ctypes

import pytest
import torch

import paper_2508_16905_amd as ta
from workloads.configs import _DEFAULT_HYPER

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("chunks", [3, 512, 513, 640, 641, 768, 1200, 1201])
@pytest.mark.parametrize("sized,k", [(8, 2), (8, 5), (8, 8), (7, 6), (6, 3), (5, 2)])
def test_same_bits_from_both(sized, k, chunks):
    first = max(1, chunks // 2)
    numels = [first * 4096 - 5, (chunks - first - 2) * 4096 + 1, 100] if chunks > 8 else [4096, 4095, 777]
    assert sum(-(-n // 4096) for n in numels) == chunks
    gen = torch.Generator(device=DEV).manual_seed(k)
    us, hus = [], []
    for n in numels:
        stride = -(-n // 4) * 4
        us.append(torch.randn(k, stride, generator=gen, device=DEV))
        hus.append(torch.randn(1, stride, generator=gen, device=DEV) + 1e-4 * torch.randn(k, stride, generator=gen, device=DEV))
    own = [u.clone() for u in us]
    vec = (ta.PowerTensor * len(numels))()
    for v, u, hu in zip(vec, us, hus):
        v.u, v.hu, v.stride = u.data_ptr(), hu.data_ptr(), u.shape[1]
    info = torch.zeros(len(numels), ctypes.sizeof(ta.PowerInfo) // 4, device=DEV)
    ta.triaccel_power_iter_static(vec, numels, k, info.data_ptr(), torch.cuda.current_stream().cuda_stream)
    opt = ta.TriAccel(dict(_DEFAULT_HYPER, power_k=sized), [torch.zeros(n, device=DEV) for n in numels])
    opt.power_iter(own, hus, k, False)
    state = opt.power_state()
    torch.cuda.synchronize()
    for l, n in enumerate(numels):
        assert torch.equal(us[l].view(torch.int32), own[l].view(torch.int32)), (l, n)
        assert list(state[l].rayleigh) == info[l, :8].tolist() and list(state[l].resid) == info[l, 8:16].tolist()
        assert list(state[l].hnorm) == info[l, 16:24].tolist()
    opt.close()
