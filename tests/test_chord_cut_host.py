"""The chord cutter (csrc/apc_cut.h, the source the kernels compile) built for the host."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    out = tmp_path_factory.mktemp("shim") / "libcut.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-o", str(out),
                           os.path.join(ROOT, "tests", "cut_host_shim.cpp")])
    L = C.CDLL(str(out))
    L.shim_cut.restype = C.c_longlong
    L.shim_cut.argtypes = [C.c_double, C.c_double, C.c_double, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p, C.c_int]

    def run(t_near, step, max_chord, at, keep=1):
        at = np.ascontiguousarray(at, dtype=np.float64)
        pieces, ends = np.zeros(len(at) - 1, dtype=np.int64), np.zeros(keep)
        n = L.shim_cut(t_near, step, max_chord, at.ctypes.data, len(at) - 1, pieces.ctypes.data, ends.ctypes.data,
                       keep)
        assert n == pieces.sum()
        return pieces, ends

    return run


def test_a_chord_too_long_to_cut_is_one_piece_and_the_others_are_cut(cut):
    """Chords of 2, 1000, 3, 0.25 and 1000 units on a lattice of 1/8 whose longest chord that is cut has 100: the
    others of the segment have a piece per lattice interval they meet."""
    at = np.cumsum([0.05, 2.0, 1000.0, 3.0, 0.25, 1000.0, 0.5])
    pieces, _ = cut(0.0, 0.125, 100.0, at)
    inside = np.floor(at / 0.125).astype(int)
    want = inside[1:] - inside[:-1] + 1  # (no end is a lattice point)
    want[[1, 4]] = 1
    assert pieces.tolist() == want.tolist()
