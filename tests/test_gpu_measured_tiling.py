"""The z-chunk of the measured march of a lattice stepped by two-step passes is
its own, not the pass's: diagnostics (whose sums depend on the tiling in their
last bits) are bitwise those of a lattice with that tiling, for a tuning entry
and for a tiling set by hand, through ah_measure and ah_step_measured."""
import numpy as np
import pytest

from helpers import same_record
from inputs import random_state

pytestmark = pytest.mark.gpu


@pytest.fixture
def ah():
    import paper_2005_14454_amd as ah
    ah.tune_clear()
    yield ah
    ah.tune_clear()


@pytest.mark.parametrize("precision,N,zchunk,own", [
    ("fp64", 96, 14, 7),
    ("fp64", 128, 32, 16),
    ("fp64", 128, 128, 16),
    ("fp32", 128, 32, 16),
    ("fp64", 40, 40, 2),
    ("fp32", 64, 16, 2),
])
def test_measured_march_has_its_own_zchunk(ah, precision, N, zchunk, own):
    gp = ah.Params(N=N, precision=precision, m=1.0)
    st = random_state(N, seed=N)
    if precision == "fp32":
        st = st.astype(np.float32).astype(np.float64)

    def records(*config):
        with ah.Lattice(gp) as lat:
            if config:
                lat.set_step_config(*config)
            lat.set_state(st, 4)
            return [lat.measure()] + lat.step_measured(5, 4) + [lat.measure()]

    want = records("tile", (32, 8), own)
    assert len(want) == 4
    got = [records("tile2", (32, 8), zchunk)]
    ah.tune_set(gp, (32, 8), zchunk, kernel="tile2")
    got.append(records())
    for series in got:
        for a, b in zip(series, want):
            assert same_record(a, b), (precision, N, zchunk)
