"""Gathers and windings through the pinned staging memory at the counts where
the number of pieces changes: one piece in the record memory, one in a handle's
own, several with a full or a ragged last one."""
import numpy as np
import pytest

from helpers import both_params
from inputs import random_state

pytestmark = pytest.mark.gpu

RECORDS, OWN = 128 << 10, 512 << 10  # bytes of the record memory, and of a small handle's staging memory


def _counts(each):
    def fits(b):
        return b // each // 32 * 32
    piece = fits(OWN // 3 // 256 * 256)
    out = {1, 31, 33, 70000}
    for n in (fits(RECORDS), fits(OWN), piece, 2 * piece, 3 * piece, 4 * piece):
        out |= {n - 1, n, n + 1}
    return sorted(out)


@pytest.mark.parametrize("precision,each", [("fp64", 88), ("fp32", 48)])
def test_gather_counts(precision, each):
    import paper_2005_14454_amd as ah
    N = 12
    st = random_state(N, seed=3)
    if precision == "fp32":
        st = st.astype(np.float32).astype(np.float64)
    gp = ah.Params(N=N, precision=precision)
    rng = np.random.default_rng(4)
    with ah.Lattice(gp) as grown:
        grown.set_state(st, 0)
        for n in _counts(each):  # small ones first: the record memory, then the handle's own
            sites = rng.integers(0, N ** 3, n)
            assert np.array_equal(grown.gather(sites), st[:, sites].T), n
            with ah.Lattice(gp) as fresh:
                fresh.set_state(st, 0)
                assert np.array_equal(fresh.gather(sites), st[:, sites].T), n


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [33, 35, 36, 39])  # 3 N^3 bytes about the record memory's and a piece's
def test_windings(oracle_mod, precision, N):
    import paper_2005_14454_amd as ah
    op, gp = both_params(oracle_mod, N, precision)
    st = random_state(N, seed=N)
    if precision == "fp32":
        st = st.astype(np.float32).astype(np.float64)
    want = oracle_mod.winding(op, st).astype(np.int8)
    with ah.Lattice(gp) as lat:
        lat.set_state(st, 0)
        assert np.array_equal(lat.winding(), want)
    with ah.Lattice(gp) as lat:  # the record memory, before a state has made the handle take its own
        lat.init(1)
        w = lat.winding()
        assert np.array_equal(w, oracle_mod.winding(op, lat.get_state()).astype(np.int8))
