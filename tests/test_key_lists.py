"""Key lists of the tensors that list all their keys: room for every wavefront's, no more of it than the tensor's
size asks for, and the device memory of a set of many small tensors as the header states it."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIST_ALL_MAX = 8192


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    d = tmp_path_factory.mktemp("key_lists")
    src, so = d / "lists.cpp", d / "liblists.so"
    src.write_text('#include "%s"\nusing namespace triaccel;\n'
                   'extern "C" void lists(int64_t n, uint32_t* o) {\n'
                   '  const KeyLists k = key_lists(n);\n'
                   '  o[0] = k.list_all; o[1] = k.sub_cap; o[2] = k.over_cap; o[3] = k.entries;\n}\n'
                   % os.path.join(ROOT, "paper_2508_16905_amd", "csrc", "common.h"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", str(so), str(src)], check=True)
    L = C.CDLL(str(so))
    L.lists.argtypes = [C.c_int64, C.c_void_p]

    def call(n):
        out = (C.c_uint32 * 4)()
        L.lists(n, out)
        return tuple(out)

    return call


def wavefront_elements(n, chunk, wave):
    """Elements of wavefront `wave` (of 4) of a chunk: 256 in each of the chunk's 4 rows of 1024."""
    return sum(min(max(n - (chunk * 4096 + row * 1024 + wave * 256), 0), 256) for row in range(4))


def test_every_wavefront_has_room_for_all_its_keys(lists):
    for n in range(1, LIST_ALL_MAX + 1):
        list_all, sub_cap, _, entries = lists(n)
        assert list_all
        for chunk in range((n + 4095) // 4096):
            for wave in range(4):
                mine = wavefront_elements(n, chunk, wave)
                assert mine <= sub_cap
                assert mine == 0 or (chunk * 4 + wave + 1) * sub_cap <= entries
        # 16 bytes per element in all, entries being 8 bytes
        assert entries <= 2 * n


def test_longer_tensors_have_short_lists_and_an_overflow_list(lists):
    for n in (LIST_ALL_MAX + 1, 12345, 262143, 262144, 262145, 1 << 30):
        cap = min(n, 262144)
        assert lists(n) == (0, (cap + 63) // 64, cap, 64 * ((cap + 63) // 64) + cap)


@pytest.mark.gpu
@pytest.mark.parametrize("numel,count", [(10, 6000), (300, 4000), (4096, 2000), (4097, 2000), (100003, 200)])
def test_workspace_of_many_small_tensors(numel, count):
    import torch

    import paper_2508_16905_amd as ta
    from workloads.configs import _DEFAULT_HYPER

    arena = torch.zeros(4 * numel + 16, dtype=torch.uint8, device="cuda")  # never read: no step is made
    config = ta.binding.Config.from_hyper(_DEFAULT_HYPER)

    def table(n):
        t = ta.binding.Tensor()
        t.param = t.grad = t.curv = t.mom = t.mask = arena.data_ptr()
        t.numel, t.grad_dtype, t.param_dtype = numel, ta.FP32, ta.FP32
        return [t] * n

    ta.binding.triaccel_destroy(ta.binding.triaccel_init(config, table(2)))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    handle = ta.binding.triaccel_init(config, table(count))
    used = before - torch.cuda.mem_get_info()[0]
    ta.binding.triaccel_destroy(handle)
    chunks = (numel + 4095) // 4096
    # include/triaccel.h: per tensor 20 KB and 16 bytes per element, 48 bytes per chunk; "a few MB" besides
    assert used <= count * (20 * 1024 + 16 * numel + 48 * chunks) + (4 << 20), (used, count)
