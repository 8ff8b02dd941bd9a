"""Steps recorded into a HIP graph and replayed between other calls on the same
handle.  The graph holds the buffers its steps were recorded on, so whatever
passes the handle takes by itself, an even number of plain steps has to leave
the snapshot in them, and a new snapshot (ah_set_state, ah_init) has to go
there: with the automatic configuration, a two-step entry of the tuning table
and a change of configuration in between, every replay gives bitwise the fields
that it gives on a handle that only takes single steps.
"""
import numpy as np
import pytest

from inputs import random_state

pytestmark = pytest.mark.gpu

N = 66  # two-step passes in both precisions


@pytest.fixture
def ah():
    import paper_2005_14454_amd as ah
    ah.tune_clear()
    yield ah
    ah.tune_clear()


def _states(precision):
    out = [random_state(N, seed=s) for s in (41, 42)]
    return [st.astype(np.float32).astype(np.float64) for st in out] if precision == "fp32" else out


def _follow(ah, gp, states, config, warm, recorded):
    """Fields after every replay and call of one program."""
    import torch
    s = torch.cuda.Stream()
    got = []
    with ah.Lattice(gp, stream=s) as lat:
        if config in ("tile", "tile, then auto"):
            lat.set_step_config("tile")
        lat.set_state(states[0], 1)
        lat.step(warm)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            lat.step(recorded)
        if config == "tile, then auto":
            lat.set_step_config("auto")

        def replay():
            with torch.cuda.stream(s):  # behind the handle's own work
                g.replay()
            torch.cuda.synchronize()
            got.append(lat.get_state())

        replay()
        for n in (2, 6, 4):  # steps between replays
            lat.step(n)
            replay()
        lat.winding()        # borrows the idle buffers
        replay()
        lat.set_state(states[1], 1)
        replay()
        lat.step(2)
        lat.init(5)
        replay()
        lat.step_measured(5, 5)  # moves the snapshot; the next call brings it back
        lat.set_state(states[0], 3)
        replay()
        replay()
    return got


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("warm,recorded", [(0, 2), (2, 2), (6, 4), (4, 6)])
@pytest.mark.parametrize("config", ["auto", "table", "tile, then auto"])
def test_replays_between_calls(ah, precision, warm, recorded, config):
    gp = ah.Params(N=N, precision=precision, m=2.0, s_late=1.0, eta_switch=1.45, eta_ref=3.0)
    states = _states(precision)
    want = _follow(ah, gp, states, "tile", warm, recorded)
    if config == "table":
        ah.tune_set(gp, (32, 8), 0, kernel="tile2")
    got = _follow(ah, gp, states, config, warm, recorded)
    for k, (a, b) in enumerate(zip(got, want)):
        assert np.array_equal(a, b), (k, precision, warm, recorded, config)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_recorded_start(ah, precision):
    """A recorded ah_init puts the start where the steps after it find it."""
    import torch
    gp = ah.Params(N=N, precision=precision)
    out = []
    for config in ("tile", "auto"):
        s = torch.cuda.Stream()
        with ah.Lattice(gp, stream=s) as lat:
            lat.set_step_config(config)
            lat.init(1)
            lat.step(2)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                lat.init(9)
            got = []
            for n in (0, 2, 4):
                lat.step(n)
                with torch.cuda.stream(s):
                    g.replay()
                torch.cuda.synchronize()
                got.append(lat.get_state())
            out.append(got)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert np.array_equal(out[1][0], out[1][2])
