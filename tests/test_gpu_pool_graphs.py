"""The pool's graphs: one is captured for each set of nodes that has work in a
replay, and used again for every later replay with that set, through admissions
and releases that fit the layout; past 64 of them they start anew.  The sets
follow from the lattices' step counts, so their number is known beforehand."""
import numpy as np
import pytest

from helpers import run_alone, same_record

pytestmark = pytest.mark.gpu


@pytest.fixture
def ah():
    import paper_2005_14454_amd as ah
    ah.tune_clear()
    yield ah
    ah.tune_clear()


def _node(k, nsteps, every, two):
    """What a replay does to a lattice at step k, and the steps it advances."""
    def due(s):
        return s == nsteps or (s < nsteps and every > 0 and s % every == 0)
    if k > nsteps:
        return None, 0
    if due(k):
        return "measured", 1
    if two and k + 1 < nsteps and not due(k + 1):
        return "two", 2
    return "single", 1


def _sets(schedule, replays):
    """Sets of nodes of each replay; schedule: (first replay, nsteps, every, node of each kind)."""
    at = [0] * len(schedule)
    out = []
    for r in range(replays):
        s = set()
        for j, (first, nsteps, every, nodes) in enumerate(schedule):
            if r < first:
                continue
            kind, n = _node(at[j], nsteps, every, "two" in nodes)
            if kind:
                s.add(nodes[kind])
                at[j] += n
        if s:
            out.append(frozenset(s))
    return out


def _captures(sets, most=64):
    held, n = set(), 0
    for s in sets:
        if s not in held:
            if len(held) >= most:
                held.clear()
            held.add(s)
            n += 1
    return n


def test_graphs_are_used_again(ah):
    p = ah.Params(N=16, precision="fp32", m=1.0)
    nodes = {"measured": "m", "single": "s", "two": "t"}
    plan = [(5 * j, 12, every, nodes) for j, every in enumerate((4, 4, 0, 3, 4, 5, 0, 4))]
    sets = _sets(plan, 60)
    assert 3 <= _captures(sets) <= 7 < len(sets)
    with ah.Pool(hbm_budget=256 << 20, max_slots=8) as pool:
        seen = []
        for r in range(60):
            for j, (first, nsteps, every, _) in enumerate(plan):
                if first == r:
                    assert pool.submit(p, j, nsteps, every) is not None
            pool.advance(1)
            for rid in pool.poll():
                pool.results(rid)
            seen.append(pool.graph_counts())
        assert seen[-1] == (1, _captures(sets))
        assert pool.stats()["graph_captures"] == 1
        # the same cadences again capture nothing
        for j in range(2):
            pool.submit(p, j, 12, 4)
        pool.advance(14)
        assert len(pool.poll()) == 2
        assert pool.graph_counts() == seen[-1]


def test_more_sets_than_are_held(ah):
    """Ten lattices of as many tile shapes and cadences: over 64 sets of nodes,
    each run's fields and series still those of the lattice alone."""
    entries = [  # precision, N, table entry, nodes of the single step and of the two-step pass
        ("fp32", 8, "tile", (64, 8), (64, 8)), ("fp32", 9, "tile", (64, 4), (64, 8)), ("fp32", 10, "tile", (32, 8), (64, 8)),
        ("fp32", 11, "tile", (128, 4), (64, 8)), ("fp32", 12, "tile", (128, 8), (64, 8)),
        ("fp32", 13, "tile2", (32, 8), (32, 8)), ("fp32", 14, "tile2", (64, 4), (64, 4)),
        ("fp64", 8, "tile", (64, 8), None), ("fp64", 9, "tile2", (32, 8), (32, 8)), ("fp64", 10, "tile2", (64, 4), (64, 4)),
    ]
    reqs, plan = [], []
    for j, (prec, N, kernel, one, two) in enumerate(entries):
        gp = ah.Params(N=N, precision=prec, m=1.0)
        ah.tune_set(gp, one, 0, kernel=kernel)
        nodes = {"measured": ("m", prec), "single": ("s", prec, one)}
        if two:
            nodes["two"] = ("t", prec, two)
        nsteps, every = 300 + j, (2, 4, 6, 8, 10, 14, 18, 2, 6, 12)[j]
        reqs.append((gp, 30 + j, nsteps, every))
        plan.append((0, nsteps, every, nodes))
    replays = 319
    sets = _sets(plan, replays)
    assert len(set(sets)) > 64 and _captures(sets) > len(set(sets))  # some are captured again
    with ah.Pool(hbm_budget=128 << 20, max_slots=10) as pool:
        ids = [pool.submit(*r) for r in reqs]
        cfgs = [pool.step_config(i) for i in ids]
        for _ in range(replays // 11):
            pool.advance(11)
        assert sorted(pool.poll()) == sorted(ids)
        assert pool.graph_counts() == (1, _captures(sets))
        states = [pool.get_state(i) for i in ids]
        series = [pool.results(i) for i in ids]
    ah.tune_clear()
    for (gp, seed, nsteps, every), cfg, st, ser in zip(reqs, cfgs, states, series):
        want, records = run_alone(gp, seed, nsteps, every, cfg["tile"], cfg["zchunk"])
        assert np.array_equal(st, want), (gp.precision, gp.N)
        assert len(ser) == len(records) and all(same_record(a, b) for a, b in zip(ser, records)), (gp.precision, gp.N)
