"""D2Q9 with half storage takes many steps per launch as every other scheme:
the source on strip and bundle edges, in the sponge and on the seam, and grids
shorter than a launch's halo, with the bits of one step per launch; and replayed
graphs on grids of the wide shape."""
import numpy as np
import pytest
import torch

from paper_1704_03172_amd import inputs, lbwave
from tests.harness import FIELDS, run_gpu

pytestmark = pytest.mark.gpu

NSTEPS = 27


def case(nx, ny, collision, source):
    rng = np.random.default_rng(nx + ny)
    rho, jx, jy = inputs.random_fields(nx, ny, seed=nx)
    rec = np.array([(x, y) for y in sorted({0, ny // 2, ny - 1}) for x in range(0, nx, 1 + nx // 90)] + [source], dtype=np.int32)
    return {"nx": nx, "ny": ny, "q": 9, "collision": collision, "tau": 0.5, "s": [1, 1, 1, 2, 2, 2, 1, 1, 2],
            "c2": rng.uniform(0.05, 0.45, (ny, nx)), "rho0": rho, "jx0": jx, "jy0": jy, "nsteps": NSTEPS,
            "sponge_width": 3 if min(nx, ny) > 6 else 0, "sponge_sigma_max": 0.1, "source": source,
            "wavelet": inputs.ricker_wavelet(NSTEPS + 1, 0.1), "receivers": rec}


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("nx,ny,source", [(700, 45, (47, 3)), (700, 45, (48, 4)), (700, 45, (0, 0)), (700, 45, (699, 44)),
                                          (481, 1, (240, 0)), (113, 5, (112, 2)), (33, 260, (31, 12)), (1, 40, (0, 39))])
def test_half_storage_d2q9(collision, nx, ny, source):
    c = case(nx, ny, collision, source)
    one = run_gpu(c, "f16s", steps_per_launch=1)
    many = run_gpu(c, "f16s")
    assert np.isfinite(one["traces"]).all() and np.abs(one["traces"]).max() > 0
    np.testing.assert_array_equal(one["traces"], many["traces"])
    for f in FIELDS:
        np.testing.assert_array_equal(one["fields"][f], many["fields"][f])


@pytest.mark.parametrize("q,precision", [(5, "f32"), (5, "f64"), (5, "f16s"), (9, "f64")])
def test_graphs_of_the_wide_shape(q, precision):
    nx, ny, calls = 1301, 619, (70, 35, 64)
    c = dict(case(nx, ny, "bgk", (96, 7)), q=q)
    out = []
    for chunk in (0, 32):
        g = lbwave.Grid(nx, ny, lattice=q, precision=precision, sponge_width=9, sponge_sigma_max=0.1, trace_capacity=sum(calls) + 1,
                        max_receivers=len(c["receivers"]), stream=torch.cuda.Stream())
        g.set_medium(c["c2"])
        g.set_state(c["rho0"], c["jx0"], c["jy0"])
        g.set_source(96, 7, 1e-2 * inputs.ricker_wavelet(sum(calls) + 1, 0.02))
        g.record(c["receivers"], fields=FIELDS)
        g.record_sum_rho()
        if chunk:
            g.set_graph(chunk)
        got = []
        for n in calls:   # the caller's work and a wait between the replays
            g.step(n)
            with torch.cuda.stream(g.stream):
                got += [g.field(f).clone() for f in FIELDS]
            g.sync()
        out.append(got + [g.traces, g.sum_rho])
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and a.abs().max() > 0
        assert torch.equal(a, b)
