"""The workspace has room for the partial sums of rho (FP64; one per row, strip
of at most 128 columns and step) of launches of as many steps as lb_blocked_steps
promises, at any size.  CPU only."""
import pytest

from paper_1704_03172_amd import lbwave


@pytest.mark.parametrize("precision,word", [("f32", 4), ("f64", 8)])
@pytest.mark.parametrize("n", [512, 1448, 1449, 2048, 4096])
def test_partial_sums_of_the_promised_steps_fit(precision, word, n):
    kw = dict(nx=n, ny=n, precision=precision)
    steps = lbwave.blocked_steps(**kw)
    populations = 2 * 5 * (n * n + 1024) * word   # rounded up to 256 elements each
    rest = lbwave.workspace_bytes(**kw) - populations - n * n * word
    assert rest >= steps * n * -(-n // 128) * 8, (rest, steps)
