"""Which kernel a round of the RoPElite search runs, and what workspace it asks for.  search_plan.hpp itself, compiled for the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_01586_amd", "csrc")


class Layout(ctypes.Structure):
    _fields_ = [(n, ctypes.c_size_t) for n in ("kp", "partial", "emask", "arrived", "res", "least", "total")] + [
        (n, ctypes.c_int) for n in ("n_tiles", "keys", "n_items")] + [("blocks", ctypes.c_bool), ("keep", ctypes.c_bool)]


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "p.cpp").write_text('#include "search_plan.hpp"\n'
                             'extern "C" void plan(long T, int n_h, size_t room, ekv::SearchLayout* out) { *out = ekv::search_layout(T, n_h, room); }\n'
                             'extern "C" size_t size() { return sizeof(ekv::SearchLayout); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "p.cpp"), "-o", str(d / "p.so")], check=True)
    lib = ctypes.CDLL(str(d / "p.so"))
    lib.size.restype = ctypes.c_size_t
    assert lib.size() == ctypes.sizeof(Layout)

    def of(T, n_h, room=None):
        out = Layout()
        lib.plan(ctypes.c_long(T), n_h, ctypes.c_size_t(0), ctypes.byref(out))
        lib.plan(ctypes.c_long(T), n_h, ctypes.c_size_t(out.total if room is None else room), ctypes.byref(out))
        return out
    return of


# measured at 128 or 64 dims: the one faster than the other by four per cent and more
@pytest.mark.parametrize("n_h,T", [(32, 176), (32, 192), (64, 128), (64, 144), (64, 192), (40, 200), (40, 224), (16, 240), (1, 1000),
                                   (32, 160), (24, 176), (24, 200), (48, 112), (28, 176), (52, 128),
                                   (8, 320), (32, 240), (32, 512), (32, 1000), (64, 640), (32, 1280)])
def test_samples_that_take_the_blocks(layout, n_h, T):
    assert layout(T, n_h).blocks


@pytest.mark.parametrize("n_h,T", [(32, 96), (64, 96), (32, 112), (32, 128), (40, 128), (20, 160), (12, 160), (20, 200), (32, 200), (32, 224),
                                   (20, 224), (32, 1536), (64, 1000), (48, 144), (28, 160), (36, 144)])
def test_samples_that_take_the_rounds(layout, n_h, T):
    assert not layout(T, n_h).blocks


@pytest.mark.parametrize("n_h", [1, 5, 8, 20, 32, 40, 64, 257])
def test_workspace_grows_with_the_sample_and_holds_what_runs(layout, n_h):
    before = layout(1, n_h)
    for T in range(1, 1600):
        L = layout(T, n_h)
        assert L.total >= before.total and L.least >= before.least and L.total >= L.least
        tight = layout(T, n_h, L.least)
        assert not tight.blocks and not tight.keep and tight.res <= L.least
        kept = L.n_items * n_h * 16 * 1024 if L.blocks else L.n_tiles * (L.n_tiles + 1) // 2 * n_h * 1024 if L.keep else 0
        assert L.res + kept <= L.total
        assert L.partial + n_h * L.n_items * 64 * 4 <= L.emask
        before = L
