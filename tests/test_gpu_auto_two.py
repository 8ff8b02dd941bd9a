"""An automatic step configuration takes two plain steps in one pass: FP32 at
every size, FP64 above 64 sites a side.  The rule against the general path,
explicit single steps: bitwise the same fields on the smallest lattices, on
both sides of the threshold and where the pass's FP32 tile changes from 32 x 8
to 64 x 8, for even and odd runs, with measured steps between them, alone and
in a pool.
"""
import numpy as np
import pytest

from helpers import run_alone, same_record
from inputs import random_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    import paper_2005_14454_amd as ah
    return ah


def _params(ah, N, precision):
    # every step has its own kick coefficients
    return ah.Params(N=N, precision=precision, m=2.0, s_early=0.0, s_late=1.0, eta_switch=1.45,
                     damp_gamma=2.0, eta_damp=1.25, eta_ref=3.0)


def _state(N, precision):
    st = random_state(N, seed=300 + N)
    return st.astype(np.float32).astype(np.float64) if precision == "fp32" else st


def _run(ah, gp, st, single, pieces):
    with ah.Lattice(gp) as lat:
        if single:
            lat.set_step_config("tile")
        else:
            assert lat.get_step_config()["kernel"] == "tile"
        lat.set_state(st, 1)
        for n in pieces:
            lat.step(n)
        return lat.get_state(), lat.step_index


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [4, 5, 24, 47, 64, 65, 75, 97, 110, 131])
def test_automatic_passes_equal_single_steps(ah, precision, N):
    gp = _params(ah, N, precision)
    st = _state(N, precision)
    for pieces in ((6,), (5, 1, 3)):
        got, n = _run(ah, gp, st, False, pieces)
        want, m = _run(ah, gp, st, True, pieces)
        assert n == m
        assert np.array_equal(got, want), (precision, N, pieces)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [9, 66, 112])
def test_automatic_evolve_equals_single_steps(ah, precision, N):
    gp = _params(ah, N, precision)
    st = _state(N, precision)
    out = []
    for single in (False, True):
        with ah.Lattice(gp) as lat:
            if single:
                lat.set_step_config("tile")
            lat.set_state(st, 1)
            series = lat.step_measured(9, 4)
            out.append((lat.get_state(), series))
    assert np.array_equal(out[0][0], out[1][0])
    assert len(out[0][1]) == len(out[1][1]) > 0
    for a, b in zip(out[0][1], out[1][1]):
        assert repr(a) == repr(b)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_pool_passes_equal_single_steps(ah, precision):
    reqs = [(ah.Params(N=N, precision=precision, m=2.0), 20 + N, 9, every)
            for N, every in ((40, 0), (65, 4), (78, 0), (78, 3))]
    with ah.Pool(hbm_budget=1 << 30, max_slots=8) as pool:
        ids = [pool.submit(*r) for r in reqs]
        cfgs = [pool.step_config(i) for i in ids]
        pool.advance(10)
        assert sorted(pool.poll()) == sorted(ids)
        for (p, seed, n, every), rid, cfg in zip(reqs, ids, cfgs):
            st, ser = run_alone(p, seed, n, every, cfg["tile"], cfg["zchunk"])
            assert np.array_equal(pool.get_state(rid, p.N), st), (precision, p.N)
            got = pool.results(rid)
            assert len(got) == len(ser) and all(same_record(a, b) for a, b in zip(got, ser))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_captured_steps_replay(ah, precision):
    """Two plain steps recorded into a HIP graph can be replayed, as single
    steps can: the buffers are back where they were after each replay."""
    import torch
    N = 66
    gp = _params(ah, N, precision)
    st = _state(N, precision)
    out = []
    for single in (False, True):
        s = torch.cuda.Stream()
        with ah.Lattice(gp, stream=s) as lat:
            if single:
                lat.set_step_config("tile")
            lat.set_state(st, 1)
            lat.step(2)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                lat.step(2)
            got = []
            for _ in range(3):
                g.replay()
                torch.cuda.synchronize()
                got.append(lat.get_state())
            out.append(got)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert not np.array_equal(out[0][0], out[0][2])


@pytest.mark.parametrize("chunk", [1, 3, 20])
def test_pool_replays_hold_every_node_with_work(ah, chunk):
    """A replay leaves out nodes without work, by the host's own count of the
    steps: requests of every short length and cadence, in both precisions,
    joining while others run, give the series and fields of a lattice alone,
    and are done on the host's count when they are on the device's."""
    P = ah.Params
    reqs = [(P(N=8 + 2 * (k % 3), precision="fp64" if k % 4 == 1 else "fp32", m=1.0), 40 + k, n, every)
            for k, (n, every) in enumerate((n, e) for n in (0, 1, 2, 3, 7) for e in (0, 1, 2, 5))]
    got = {}
    with ah.Pool(hbm_budget=256 << 20, max_slots=len(reqs)) as pool:
        waiting, ids = list(enumerate(reqs)), {}
        for _ in range(200):
            if waiting:
                k, r = waiting.pop(0)
                ids[pool.submit(*r)] = k
            pool.advance(chunk)
            pool.synchronize()
            for rid in pool.poll_async():
                k = ids[rid]
                p, _, n, _ = reqs[k]
                assert pool.progress(rid) == (n, n)
                cfg = pool.step_config(rid)
                state = pool.get_state(rid, p.N)
                got[k] = (cfg, state, pool.results(rid))
            if len(got) == len(reqs):
                break
        assert len(got) == len(reqs)
    for k, (p, seed, n, every) in enumerate(reqs):
        cfg, state, series = got[k]
        st, ser = run_alone(p, seed, n, every, cfg["tile"], cfg["zchunk"])
        assert np.array_equal(state, st), (p, n, every)
        assert len(series) == len(ser) and all(same_record(a, b) for a, b in zip(series, ser)), (p, n, every)


@pytest.mark.parametrize("precision,sizes", [
    ("fp32", (66,)), ("fp32", (8, 9, 66)), ("fp32", (24,) * 20 + (40,) * 9 + (51, 90)), ("fp64", (65, 66, 90, 130)),
])
def test_pool_work_lists_hold_every_tile(ah, precision, sizes):
    """Two-step z-chunks follow from what is in the pool, and the tiles' runs
    are dealt to the XCDs by load: whatever the mix, every site is stepped
    once (the fields of a lattice alone)."""
    reqs = [(ah.Params(N=N, precision=precision, m=1.0), 70 + k, 5, 0) for k, N in enumerate(sizes)]
    with ah.Pool(hbm_budget=2 << 30, max_slots=40) as pool:
        ids = [pool.submit(*r) for r in reqs[:-1]]
        pool.advance(1)
        ids.append(pool.submit(*reqs[-1]))
        pool.advance(7)
        assert sorted(pool.poll()) == sorted(ids)
        for k, (p, seed, n, _) in enumerate(reqs):
            if k % 5 and k < len(reqs) - 3:
                continue
            with ah.Lattice(p) as lat:
                lat.set_step_config("tile")
                lat.init(seed)
                lat.step(n)
                assert np.array_equal(pool.get_state(ids[k], p.N), lat.get_state()), (k, p.N)
