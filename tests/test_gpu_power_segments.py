"""Power iteration on either side of the rule that gives every chunk its own segment: both entry points against ordered
Gram-Schmidt in 64 bits.  The products are well conditioned (normal entries, many more elements than vectors), so the
stored value is the rounding of the fp64 result, 6e-8 of it, or the next one; norms likewise."""
import ctypes

import pytest
import torch

import paper_2508_16905_amd as ta
from workloads.configs import _DEFAULT_HYPER

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("entry", ["handle", "static"])
@pytest.mark.parametrize("k,chunks", [(5, 768), (5, 769), (8, 512), (8, 513), (1, 768), (3, 3), (6, 1200), (6, 1201), (7, 640), (8, 641)])
def test_segments_of_one_chunk_and_of_four(k, chunks, entry):
    first = max(1, chunks // 2)
    numels = [first * 4096 - 5, (chunks - first - 3) * 4096 + 1, 4096, 100] if chunks > 8 else [4096, 4095, 777]
    assert sum(-(-n // 4096) for n in numels) == chunks
    gen = torch.Generator(device=DEV).manual_seed(k)
    us, hus = [], []
    vec = (ta.PowerTensor * len(numels))()
    for v, n in zip(vec, numels):
        stride = -(-n // 4) * 4
        us.append(torch.randn(k, stride, generator=gen, device=DEV))
        hus.append(torch.randn(k, stride, generator=gen, device=DEV))
        v.u, v.hu, v.stride = us[-1].data_ptr(), hus[-1].data_ptr(), stride
    if entry == "static":
        info = torch.zeros(len(numels), ctypes.sizeof(ta.PowerInfo) // 4, device=DEV)
        ta.triaccel_power_iter_static(vec, numels, k, info.data_ptr(), torch.cuda.current_stream().cuda_stream)
        norms = info[:, 16:16 + k]
    else:
        opt = ta.TriAccel(dict(_DEFAULT_HYPER, power_k=k), [torch.zeros(n, device=DEV) for n in numels])
        opt.power_iter(us, hus, k, False)
        norms = torch.tensor([list(x.hnorm[:k]) for x in opt.power_state()], device=DEV)
        opt.close()
    for l, (u, hu, n) in enumerate(zip(us, hus, numels)):
        q = []
        for j in range(k):
            w = hu[j, :n].double()
            assert abs(float(norms[l, j]) / float(w.norm()) - 1) < 2e-7
            for _ in range(2):
                for p in q:
                    w = w - (p @ w) * p
            q.append(w / w.norm())
        want = torch.stack(q)
        assert float((u[:, :n].double() - want).abs().max() / want.abs().max()) < 2 * 2.0 ** -24 + 1e-11, (l, n)
