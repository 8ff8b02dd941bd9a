"""The fold of a lattice's diagnostics records: one block sums every record of
a measured launch, 64 records at a time and eight of those in flight.  The
z-chunk sets how many records a launch leaves: one, fewer than 64, a multiple
of 64, one past it, and more than the 512 that are in flight at once."""
import numpy as np
import pytest

from helpers import both_params
from inputs import random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,N,zchunk,records", [
    ("fp64", 8, 8, 1), ("fp64", 12, 12, 2), ("fp64", 24, 2, 36), ("fp64", 32, 2, 64), ("fp64", 40, 2, 200),
    ("fp64", 64, 2, 512), ("fp64", 68, 2, 918), ("fp32", 8, 8, 1), ("fp32", 32, 2, 64), ("fp32", 68, 8, 243),
])
def test_fold_sums_every_record(oracle_mod, precision, N, zchunk, records):
    """Sums against the oracle: exact counts; energies, R and the Gauss norms to
    1e-11 of the total energy or of themselves (FP64: ~N^3 terms of one sign,
    each within a few 1e-15; FP32 densities: 1e-6)."""
    import paper_2005_14454_amd as ah
    op, gp = both_params(oracle_mod, N, precision, m=1.0)
    tile = (32, 8)  # the measured march's
    assert -(-N // tile[0]) * -(-N // tile[1]) * -(-N // zchunk) == records
    st = random_state(N, seed=N)
    if precision == "fp32":
        st = st.astype(np.float32).astype(np.float64)
    with ah.Lattice(gp) as lat:
        lat.set_step_config("tile", tile, zchunk)
        lat.set_state(st, 3)
        got = lat.measure()
        assert lat.step_measured(1, 3)[0] == got  # the same records through the fused step
    ref = oracle_mod.measure(op, st, 3)
    tol = 1e-11 if precision == "fp64" else 1e-6
    assert got["winding_sum_abs"] == ref["winding_sum_abs"] and got["nonfinite"] == 0
    for k in ("energy", "e_kin", "e_grad", "e_pot", "e_el", "e_mag", "sum_L"):
        assert abs(got[k] - ref[k]) <= tol * ref["energy"], k
    for k in ("R", "v2_omega", "gauss_rms", "gauss_max", "gauss_rel"):
        assert abs(got[k] - ref[k]) <= 10 * tol * abs(ref[k]), k


def test_fold_counts_every_record(oracle_mod):
    """One non-finite site in each workgroup's share: the count adds over all records."""
    import paper_2005_14454_amd as ah
    N = 64
    st = random_state(N, seed=1).reshape(10, N, N, N)
    st[2, ::2, ::8, ::32] = np.inf  # Pi: one site of every 32 x 8 x 2 workgroup
    with ah.Lattice(ah.Params(N=N, precision="fp64")) as lat:
        lat.set_step_config("tile", (32, 8), 2)
        lat.set_state(st.reshape(10, -1), 0)
        assert lat.measure()["nonfinite"] == 32 * 8 * 2
