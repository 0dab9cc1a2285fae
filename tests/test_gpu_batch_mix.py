"""The batched executor against grids of their own, bit for bit, where the rounds
take different kernels and lengths: active shots of few and of many nodes
together (the shape and the steps of a round change when a shot is admitted or
retired), ticks that replay several graphs and leave a remainder, ticks of one
step."""
import numpy as np
import pytest

from paper_1704_03172_amd import inputs

pytestmark = pytest.mark.gpu

MRT5 = [1, 1, 1, 1.6, 1.3]
MRT9 = [1, 1, 1, 2, 2, 2, 1, 1, 2]
# nodes: 39 k, 0.74 M (0.78 M together), 0.82 M (1.6 M), 1.3 M (2.9 M)
SIZES = [(301, 129, 97), (617, 1203, 150), (1009, 811, 91), (1301, 977, 83)]


def shot(nx, ny, nsteps):
    rng = np.random.default_rng(nx)
    rec = np.array([(x, y) for y in (9, ny // 2, ny - 1) for x in (0, 47, 48, 95, 96, 97, nx // 2, nx - 1) if x < nx],
                   dtype=np.int32)
    return {"nx": nx, "ny": ny, "nsteps": nsteps, "c2": rng.uniform(0.05, 0.45, (ny, nx)), "src": (96, 12), "rec": rec,
            "wavelet": inputs.ricker_wavelet(nsteps + 1, 0.05)}


def alone(sh, **scheme):
    from paper_1704_03172_amd import lbwave
    g = lbwave.Grid(sh["nx"], sh["ny"], sponge_width=9, sponge_sigma_max=0.1, trace_capacity=sh["nsteps"] + 1,
                    max_receivers=len(sh["rec"]), **scheme)
    g.set_medium(sh["c2"])
    g.set_state(np.zeros((sh["ny"], sh["nx"])))
    g.set_source(sh["src"][0], sh["src"][1], sh["wavelet"])
    g.record(sh["rec"])
    g.step(sh["nsteps"])
    out = g.traces[0].cpu().numpy()
    assert np.isfinite(out).all() and np.abs(out).max() > 0
    return out


def together(shots, ticks, when, use_graph, **scheme):
    """Traces of the shots, shot i admitted before tick when[i] and retired
    after the tick that finishes it; ticks repeats."""
    from paper_1704_03172_amd import lbwave
    b = lbwave.Batch(len(shots), use_graph=use_graph, **scheme)
    out, slots, k = {}, {}, 0
    while len(out) < len(shots):
        for i, s in enumerate(shots):
            if when[i] == k:
                d = lbwave.shot_desc(s["nx"], s["ny"], s["src"], s["nsteps"], len(s["rec"]), 9, 0.1)
                slots[b.add(d, s["c2"], s["wavelet"], s["rec"])] = i
        b.tick(ticks[k % len(ticks)])
        b.sync()
        times = b.times()
        for slot in list(slots):
            i = slots[slot]
            if times[slot] >= shots[i]["nsteps"]:
                out[i] = b.remove(slot).cpu().numpy()
                del slots[slot]
        k += 1
    b.close()
    return [out[i] for i in range(len(shots))]


@pytest.mark.parametrize("scheme", [dict(), dict(collision="mrt", s=MRT5), dict(precision="f64"), dict(precision="f16s"),
                                    dict(precision="f64", lattice=9, collision="mrt", s=MRT9), dict(lattice=9)])
def test_mix_of_all_sizes(scheme):
    shots = [shot(*k) for k in SIZES]
    want = [alone(k, **scheme) for k in shots]
    for use_graph in (True, False):
        # 0.78 M nodes, then 1.6 M, then 2.9 M; the shots end at different ticks
        got = together(shots, [33, 7, 1, 40], [0, 0, 1, 2], use_graph, **scheme)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("scheme", [dict(), dict(precision="f64"), dict(lattice=9), dict(precision="f16s", lattice=9)])
def test_ticks_of_many_graphs(scheme):
    """70 steps are two or more replays and a remainder at every step count."""
    shots = [shot(301, 129, 290), shot(97, 211, 215), shot(130, 67, 141)]
    want = [alone(k, **scheme) for k in shots]
    for use_graph in (True, False):
        got = together(shots, [70], [0, 0, 1], use_graph, **scheme)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("precision", ["f32", "f64", "f16s"])
@pytest.mark.parametrize("q,collision,tau,s", [(5, "bgk", 0.5, None), (5, "bgk", 0.8, None), (5, "mrt", 0.5, MRT5),
                                               (9, "bgk", 0.5, None), (9, "mrt", 0.5, MRT9)])
def test_ticks_of_one_step(precision, q, collision, tau, s):
    """Ticks of one step, and longer ones whose remainder is one step, with
    shots of both forms of the collision, narrower and wider than a block."""
    scheme = dict(lattice=q, collision=collision, precision=precision, tau=tau, s=s)
    shots = [shot(701, 401, 23), shot(1100, 64, 14), shot(100, 30, 19)]
    want = [alone(k, **scheme) for k in shots]
    for use_graph in (True, False):
        got = together(shots, [1, 1, 17, 1], [0, 1, 0], use_graph, **scheme)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
