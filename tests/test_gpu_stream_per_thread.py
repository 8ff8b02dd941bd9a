"""A handle on hipStreamPerThread, which names another stream in each thread:
state and windings of lattices large enough for helper threads (16 MB of host
data and more) still come after the handle's own work, bitwise as on an
ordinary stream."""
import types

import numpy as np
import pytest

from inputs import random_state

pytestmark = pytest.mark.gpu

PER_THREAD = types.SimpleNamespace(cuda_stream=2)  # hipStreamPerThread


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_state_on_the_threads_stream(precision):
    import paper_2005_14454_amd as ah
    N = 66
    gp = ah.Params(N=N, precision=precision)
    out = []
    for stream in (None, PER_THREAD):
        with ah.Lattice(gp, stream=stream) as lat:
            got = []
            for seed in (1, 2):
                lat.set_state(random_state(N, seed=seed), 1)
                got.append(lat.gather_noalloc(np.arange(0, N ** 3, 977)))  # first to use the uploaded fields
                lat.step(3)
                got.append(lat.get_state())
                got.append(lat.winding())
            out.append(got)
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_windings_on_the_threads_stream(precision):
    import paper_2005_14454_amd as ah
    gp = ah.Params(N=180, precision=precision)
    out = []
    for stream in (None, PER_THREAD):
        with ah.Lattice(gp, stream=stream) as lat:
            lat.init(3)
            w = []
            for _ in range(2):
                lat.step(2)
                w.append(lat.winding())
            out.append(w)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert not np.array_equal(out[1][0], out[1][1])
