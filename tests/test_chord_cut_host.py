"""The chord cutter (csrc/apc_cut.h, the source the kernels compile) built for the host."""
import ctypes as C
import os
import subprocess
from fractions import Fraction

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


@pytest.mark.parametrize("step", [1e-3, 1.0 / 3.0 * 1e-6, 0.7e-7])
def test_cut_points_are_lattice_points_to_the_last(cut, step):
    """The last of up to 7 million cut points of a segment of 5000 chords is its lattice point t_near + k * step
    rounded once, as the first is: a unit in the last place at most."""
    t_near = -0.85
    at = np.concatenate([[-0.513], -0.5 + 0.49 * np.cumsum(np.linspace(1.0, 3.0, 5000)) / 10000.0])
    pieces, ends = cut(t_near, step, 1e9, at, keep=9)
    assert pieces.sum() > 0.48 / step
    n = int(pieces.sum())
    for e in (ends[i % 9] for i in range(n - 8, n)):
        if e in at:
            continue  # a chord's end
        k = round((Fraction(float(e)) - Fraction(t_near)) / Fraction(step))
        point = Fraction(t_near) + k * Fraction(step)
        assert abs(Fraction(float(e)) - point) <= Fraction(float(np.spacing(abs(e))))
