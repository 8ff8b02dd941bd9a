"""State I/O through the pinned staging memory: what goes in comes out, bit for
bit (FP32: rounded to FP32), for rows with and without padding, states that
fit the handle's record memory and states of many pieces with a ragged last
one, from either pair of buffers; the sites gathered one by one and the rest
of the API agree with the fields that were read."""
import numpy as np
import pytest

from inputs import random_state, sample_sites

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    import paper_2005_14454_amd as ah
    return ah


def _marked(N):
    """A state whose every value names its component and site."""
    st = np.arange(10 * N ** 3, dtype=np.float64).reshape(10, N ** 3)
    return (st + 1.0) / 1024.0 - 3.0


def _stored(st, precision):
    return st.astype(np.float32).astype(np.float64) if precision == "fp32" else st


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [4, 7, 16, 32, 33, 64, 75, 90])
def test_state_round_trip(ah, precision, N):
    a, b = _marked(N), _stored(random_state(N, seed=N), precision)
    with ah.Lattice(ah.Params(N=N, precision=precision)) as lat:
        for st in (a, b, a):
            lat.set_state(st, 2)
            assert np.array_equal(lat.get_state(), _stored(st, precision))
        # values that a conversion could change: signed zeros, subnormals, infinities, NaN
        st = b.copy()
        st[:, :8] = [0.0, -0.0, 1e-40, -1e-40, np.inf, -np.inf, np.nan, 3e38]
        lat.set_state(st, 2)
        got = lat.get_state()
        want = _stored(st, precision)
        assert np.array_equal(got, want, equal_nan=True)
        assert np.array_equal(np.signbit(got[:, :6]), np.signbit(want[:, :6]))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [10, 50, 66])
def test_state_after_steps(ah, precision, N):
    """The snapshot read and gathered is that of the buffers it is in (single
    steps swap one pair, measured steps and two-step passes the other), and
    the windings, which borrow the idle pair, leave it alone."""
    gp = ah.Params(N=N, precision=precision, m=2.0)
    st = _stored(random_state(N, seed=7), precision)
    sites = np.concatenate([sample_sites(N, 300, seed=5), [0, N ** 3 - 1]])
    many = np.arange(30000, dtype=np.int64) * 7919 % N ** 3
    with ah.Lattice(gp) as lat, ah.Lattice(gp) as ref:
        lat.set_state(st, 1)
        ref.set_state(st, 1)
        for move in ("step 1", "measured", "step 2", "step 3"):
            for q in (lat, ref):
                q.step_measured(1, 1) if move == "measured" else q.step(int(move[-1]))
            got = lat.get_state()
            w = lat.winding()
            assert np.array_equal(lat.get_state(), got), move
            assert np.array_equal(lat.winding(), w)
            assert np.array_equal(lat.gather(sites), got[:, sites].T), move
            assert np.array_equal(lat.gather(many), got[:, many].T), move
        assert np.array_equal(ref.get_state(), got)
        # a state read back and put into a fresh lattice goes on alike
        with ah.Lattice(gp) as other:
            other.set_state(got, lat.step_index)
            other.step(3)
            lat.step(3)
            assert np.array_equal(other.get_state(), lat.get_state())


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_pool_state(ah, precision):
    with ah.Pool(hbm_budget=1 << 30, max_slots=4) as pool:
        for N in (20, 70):
            gp = ah.Params(N=N, precision=precision)
            rid = pool.submit(gp, N, 5, 0)
            pool.advance(3)
            got = pool.get_state(rid, N)
            step = pool.progress(rid)[0]
            with ah.Lattice(gp) as lat:
                lat.init(N)
                lat.step(step)
                assert np.array_equal(got, lat.get_state())
