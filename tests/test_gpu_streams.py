"""A grid on a stream of its own, called from another stream: every call that
reads or fills tensors is ordered after the caller's work so far, and what it
returns is ready for the caller's later work.  The caller's stream is kept busy
for milliseconds before each call, inputs are dropped at once and their memory
used again, and the results are used without a wait on the host."""
import numpy as np
import pytest
import torch

from paper_1704_03172_amd import inputs

pytestmark = pytest.mark.gpu

NX, NY, NSTEPS = 301, 201, 60


def busy():
    big = torch.zeros(1 << 26, device="cuda")
    for _ in range(100):
        big.add_(1.0)


def late(a):
    """A tensor that gets its values only after the stream's work so far."""
    out = torch.zeros_like(a)
    busy()
    out.copy_(a)
    return out


def run(stream, wait):
    """All results of a run; wait: hand the inputs over late, use the outputs at once."""
    from paper_1704_03172_amd import lbwave
    hand = late if wait else (lambda a: a)
    rng = np.random.default_rng(3)
    dev = lambda a: torch.as_tensor(a, device="cuda", dtype=torch.float32)
    c2, rho, obs = dev(rng.uniform(0.05, 0.45, (NY, NX))), dev(inputs.random_fields(NX, NY, seed=4)[0]), \
        dev(rng.standard_normal((20, NSTEPS + 1)))
    rec = np.stack([rng.integers(0, NX, 20), rng.integers(0, NY, 20)], axis=1).astype(np.int32)
    if wait:
        busy()
    g = lbwave.Grid(NX, NY, trace_capacity=NSTEPS + 1, max_receivers=20, rho_tape=1, stream=stream)
    g.set_medium(hand(c2))
    g.set_state(hand(rho))
    again = [torch.full_like(rho, 7.0) for _ in range(3)] if wait else None   # the memory of dropped inputs
    g.set_source(100, 50, 1e-2 * inputs.ricker_wavelet(NSTEPS + 1, 0.1))
    if wait:
        busy()
    traces, sums = g.record(rec), g.record_sum_rho()
    g.step(NSTEPS - 20)
    out = [g.field("rho").clone()]
    blob = g.get_state()
    g.set_raw_state(hand(blob))       # ends the tape, as any state of another run
    out.append(g.field("jx").clone())
    g.set_state(hand(rho))
    g.step(NSTEPS)
    phi, res = g.misfit(hand(obs), NSTEPS)
    out += [phi.clone(), res.clone()]
    out.append(g.adjoint(hand(res), NSTEPS).clone())
    g.sync()
    torch.cuda.synchronize()
    del again
    return out + [traces.clone(), sums.clone()]


def test_calls_are_ordered_with_the_callers_stream():
    want = run(None, False)
    assert all(torch.isfinite(a).all() and a.abs().max() > 0 for a in want)
    for stream, caller in ((torch.cuda.Stream(), torch.cuda.default_stream()), (torch.cuda.Stream(), torch.cuda.Stream()),
                           (torch.cuda.default_stream(), torch.cuda.Stream())):
        torch.cuda.synchronize()
        with torch.cuda.stream(caller):
            got = run(stream, True)
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            assert torch.equal(a, b)
