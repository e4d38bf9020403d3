"""Stage 0 of the in-place 2 <-> 4-byte rewrite with its chunks side by side (plans with subtree stages):
chunk c < top is loaded in launch 0 and its new values are copied into place in the launch that
``resize_copy_launch`` names.  Replayed on the byte map of tests/test_resize_schedule.py."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from test_resize_schedule import E, REAL, SIZES, lib, replay, events, sets_with  # noqa: F401  (lib is the fixture)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def copy_launch(tmp_path_factory):
    d = tmp_path_factory.mktemp("resize_top")
    src, so = d / "top.cpp", d / "libtop.so"
    src.write_text('#include "%s"\nusing namespace triaccel;\n'
                   'extern "C" void top(uint32_t m, uint32_t t, uint32_t n, int narrowing, uint32_t* o) {\n'
                   '  const ResizePlan p = make_resize_plan(m, t, n);\n'
                   '  o[0] = p.n_stages; o[1] = p.top; o[2] = p.n_stages > 1 ? resize_copy_launch(p, narrowing != 0) : 0u;\n}\n'
                   % os.path.join(ROOT, "paper_2508_16905_amd", "csrc", "resize_schedule.h"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", str(so), str(src)], check=True)
    L = C.CDLL(str(so))
    L.top.argtypes = [C.c_uint32, C.c_uint32, C.c_uint32, C.c_int, C.c_void_p]

    def call(set_, narrowing):
        out = np.zeros(3, np.uint32)
        L.top(*set_, int(narrowing), out.ctypes.data)
        return tuple(int(v) for v in out)

    return call


def side_by_side(ev, n_chunks, top, at):
    rest = ev[ev[:, 4] != 0]
    first = [(0, 1 << 20 | c, 0, c, 0) for c in range(min(top, n_chunks))]
    last = [(at, 1 << 20 | c, 2, c, 0) for c in range(min(top, n_chunks))]
    rows = np.array(first + [tuple(r) for r in rest] + last, np.int32)
    return rows[np.argsort(rows[:, 0], kind="stable")]


@pytest.mark.parametrize("narrowing", [True, False])
def test_copies_land_on_bytes_already_loaded(lib, copy_launch, narrowing):  # noqa: F811
    for max_chunks in [s for s in SIZES if s > 128]:
        for set_ in sets_with(lib, max_chunks) + [s for s, _, _ in REAL.values() if s[0] == max_chunks]:
            n_stages, top, at = copy_launch(set_, narrowing)
            assert n_stages > 1 and 0 < at < n_stages
            for n_chunks in sorted({1, top - 1, top, top + 1, 2 * top, 2 * top + 1, max_chunks - 1, max_chunks}):
                if n_chunks > max_chunks:
                    continue
                for tail in (1, E):
                    ev = events(lib, set_, n_chunks, narrowing)
                    replay(side_by_side(ev, n_chunks, top, at), n_chunks, (n_chunks - 1) * E + tail, narrowing)


def test_a_copy_one_launch_early_is_caught(lib, copy_launch):  # noqa: F811
    for narrowing in (True, False):
        _, top, at = copy_launch((1024, 1024, 1), narrowing)
        ev = events(lib, (1024, 1024, 1), 1024, narrowing)
        with pytest.raises(AssertionError):
            replay(side_by_side(ev, 1024, top, at - 1), 1024, 1024 * E, narrowing)
