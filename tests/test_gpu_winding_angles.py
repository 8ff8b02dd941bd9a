"""Windings in the measured march where plaquette angles lie within a few 1e-4
turns of a half turn, at link phases |dx A| from small to past 100: the count
equals the sum over the winding field, and both the oracle's, as the angles
are formed, wrapped and added to the link phases in FP64 whatever the storage
precision."""
import numpy as np
import pytest

from helpers import both_params
from inputs import grid, random_state

pytestmark = pytest.mark.gpu


def _half_turn_state(N, seed, dx, top):
    """|dx A| in (top - 2 pi, top], the (x, y) plaquette angles at even x1 an odd
    number of half turns and up to 4e-4 turns more or less."""
    rng = np.random.default_rng(seed)
    st = random_state(N, seed=seed)
    V = N ** 3
    x0, x1, x2 = grid(N)
    a = rng.uniform(max(top - 1.0, 0.0), top, (3, V)) * rng.choice([-1.0, 1.0], (3, V))
    at = np.arange(V)
    xp = (x0 + 1) % N + N * (x1 + N * x2)
    yp = x0 + N * ((x1 + 1) % N + N * x2)
    even = at[x1 % 2 == 0]
    angle = np.pi + 2.0 * np.pi * rng.uniform(-4e-4, 4e-4, len(even))
    want = a[0, even] + a[1, xp[even]] - a[1, even] - angle  # of A_x at odd x1, up to whole turns
    a[0, yp[even]] = top - np.mod(top - want, 2.0 * np.pi)
    st[4:7] = a / dx
    return st


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("top", [2.0 * np.pi, 30.0, 100.0, 106.5, 1000.0])
def test_windings_at_half_turns(oracle_mod, precision, top):
    import paper_2005_14454_amd as ah
    N = 40
    op, gp = both_params(oracle_mod, N, precision)
    st = _half_turn_state(N, 11, op["dx"], top)
    if precision == "fp32":
        st = st.astype(np.float32).astype(np.float64)
    want = oracle_mod.winding(op, st)
    assert np.count_nonzero(want) > 0
    with ah.Lattice(gp) as lat:
        lat.set_state(st, 3)
        assert np.array_equal(lat.winding(), want.astype(np.int8))
        assert lat.measure()["winding_sum_abs"] == np.abs(want).sum()
        assert lat.step_measured(1, 1)[0]["winding_sum_abs"] == np.abs(want).sum()
