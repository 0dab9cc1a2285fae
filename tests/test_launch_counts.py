"""Step counts per launch that are stated outside the library against its own
rules (host functions, no GPU): what lb_blocked_steps promises is at most what a
launch may take, so that a call of n steps takes at most ceil((n - 1) / promise)
launches and one; bench.py's counts are the library's."""
import ctypes

import pytest

import bench
from paper_1704_03172_amd import lbwave

STORAGE = {"f32": 0, "f64": 1, "f16s": 2}
SIDES = (1, 30, 48, 128, 181, 182, 316, 317, 512, 565, 566, 894, 895, 1024, 1264, 1265, 1414, 1415, 1448, 1643, 1644, 2048, 2121,
         2122, 2345, 2346, 3000, 4096)


class Choice(ctypes.Structure):
    _fields_ = [("small", ctypes.c_bool), ("steps", ctypes.c_int32)]


def choose(name, precision, q, nodes):
    f = getattr(lbwave.lib(), name)
    f.restype, f.argtypes = Choice, [ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    return f(STORAGE[precision], q, nodes).steps


@pytest.mark.parametrize("q", [5, 9])
@pytest.mark.parametrize("precision", ["f32", "f64", "f16s"])
def test_counts_follow_the_library(q, precision):
    for n in SIDES:
        steps = choose("_ZN3lbw11flow_chooseEiil", precision, q, n * n)
        assert bench.steps_per_launch(n, q, precision) == steps, n
        if precision == "f32":
            assert bench.backward_steps_per_launch(n, q) == choose("_ZN3lbw19flow_adjoint_chooseEiil", precision, q, n * n), n
        for nx, ny in ((n, n), (4 * n, n), (n, 3 * n)):
            for collision in ("bgk", "mrt"):
                for cap in range(9):
                    kw = dict(nx=nx, ny=ny, lattice=q, collision=collision, precision=precision, steps_per_launch=cap,
                              s=[1, 1, 1, 2, 2, 2, 1, 1, 2][:q])
                    most = choose("_ZN3lbw11flow_chooseEiil", precision, q, nx * ny)
                    assert lbwave.blocked_steps(**kw) <= (min(most, cap) if cap else most), kw


@pytest.mark.parametrize("m,most,want", [(1, 16, 1), (2, 16, 2), (55, 16, 14), (55, 8, 8), (17, 16, 9), (3000, 16, 16), (20, 12, 10)])
def test_even_division(m, most, want):
    assert bench.even_steps(m, most) == want
    taken = launches = 0
    while taken < m:
        ns = bench.even_steps(m - taken, most)
        assert 1 <= ns <= most
        taken += ns
        launches += 1
    assert taken == m and launches == -(-m // most)
