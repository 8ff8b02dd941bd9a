"""The FP64 64 x 4 two-step pass reads the planes below its own column back from
LDS, from slots that it writes in the same phase: bitwise single steps for the
shortest chunks, a last chunk of one plane, chunks of an even and an odd number
of planes and ragged tiles."""
import numpy as np
import pytest

from inputs import random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,zchunk", [(4, 2), (5, 2), (7, 3), (9, 4), (65, 2), (66, 33), (67, 0), (130, 8), (131, 26)])
def test_column_read_back(N, zchunk):
    import paper_2005_14454_amd as ah
    gp = ah.Params(N=N, precision="fp64", m=2.0, s_late=1.0, eta_switch=1.45, eta_ref=3.0)
    st = random_state(N, seed=N)
    out = []
    for config in (("tile2", (64, 4), zchunk), ("tile", (64, 4), 0)):
        with ah.Lattice(gp) as lat:
            lat.set_step_config(*config)
            lat.set_state(st, 1)
            lat.step(4)
            out.append(lat.get_state())
    assert np.array_equal(out[0], out[1])
