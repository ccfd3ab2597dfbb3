"""CPU tests of the heap and parDijkstra logic as teams of wavefronts run it
(tests/hostmodel/lanes.h): the register forms of one wavefront, the shortcut
past an idle Resolve(0), ballots and scans, staging tiles and list sorts, which
the one-thread team of test_hostmodel.py does not pass through.  The
invariants are those of that file, and every count equals the one-thread
team's."""
import numpy as np
import pytest

import oracle
import workloads as W
from hostmodel import HostHeap, fill, kept_team, lane_order, sssp as hm_sssp
from test_hostmodel import NGRAPHS, _graphs, check_structure

LANES = [64, 256]


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("seed", range(12))
def test_random_scripts_with_deletes_vs_oracle(lanes, seed):
    d = [1, 2, 3, 4, 7, 16][seed % 6]
    cap = [5, 40, 300, 1000][seed % 4]
    maxb = [d, 3 * d, 60][seed % 3]
    h, o = HostHeap(cap, d, seed % 2, lanes), oracle.PQ(cap)
    for op in W.random_script(40, cap, maxb, [3, 50, 10 ** 9][seed % 3], 900 + seed, deletes=True):
        if op[0] == "update":
            h.bulk_update(op[1], op[2])
            o.bulk_update(op[1], op[2])
        elif op[0] == "delete":
            h.delete(op[1])
            o.delete(op[1])
        else:
            k1, v1 = h.extract_min(op[1])
            k2, v2 = o.extract_min(op[1])
            assert np.array_equal(k1, k2) and np.array_equal(v1, v2)
        assert check_structure(h, o.cur(), d)["live"] == o.size()


def both(g, src, lanes, **kw):
    rc, dist, st = hm_sssp(g, src, lanes=lanes, check_live=True, **kw)
    rc1, dist1, st1 = hm_sssp(g, src, **kw)
    assert rc == rc1 == 0
    assert st["first_bad"] == -1, st["violation"]
    assert np.array_equal(dist, oracle.dijkstra(g, src)) and np.array_equal(dist1, dist)
    for k in ("rounds", "relax", "updates", "elems", "resolves", "extracted", "levels"):
        assert st[k] == st1[k], k


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("gi", [g for g in range(NGRAPHS) if g != 6])  # (6 is a large one)
@pytest.mark.parametrize("variant", [(0, 0, 0), (1, 0, 2), (0, 1, 1), (0, 3, 2)])
def test_plain_rounds(lanes, gi, variant):
    sched, dmul, qlds = variant
    g = list(_graphs())[gi]
    both(g, (gi * 7) % g.n, lanes, d=max(1, g.max_degree()) * dmul, sched=sched, qlds=qlds)


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("gi", [0, 1, 2, 4, 5, 12, 16, 18])
@pytest.mark.parametrize("lds", [0, 40_000])
def test_speculative_rounds(lanes, gi, lds):
    """Rounds of k extractions, their lists in HBM or sorted in LDS."""
    g = list(_graphs())[gi]
    kw = dict(rule=3, kseq=[40, 1, 7, 256, 3], kmax=256, d=max(32, g.max_degree()))
    if not lds:
        both(g, 0, lanes, **kw)
        return
    rc, dist, st = hm_sssp(g, 0, **kw)
    with kept_team(lds, lanes):
        rc, dist, st2 = hm_sssp(g, 0, lanes=lanes, qlds=1, check_live=True, **kw)
    assert rc == 0 and st2["first_bad"] == -1 and np.array_equal(dist, oracle.dijkstra(g, 0))
    assert all(st2[k] == st[k] for k in ("rounds", "relax", "updates", "elems", "resolves"))


@pytest.mark.parametrize("lanes", LANES)
def test_merges_of_several_tiles(lanes):
    both(W.random_graph(3000, 30000, 0, 10 ** 6, 5), 0, lanes, rule=1, kfix=200, kmax=256, d=150, qlds=0)
    both(W.random_graph(1500, 9000, 0, 10 ** 6, 5), 0, lanes, d=40, qlds=1)


@pytest.mark.parametrize("lanes", LANES)
def test_a_team_goes_from_query_to_query(lanes):
    """As the test of this name with one thread: queries with a staging area
    after their one LDS level, then queries with two levels in its place, and
    merges in HBM that are large enough for one."""
    d = 32
    gs = [W.random_graph(n, 5 * n, 0, 10 ** 6, 7 + n) for n in (14 * lanes, 16 * lanes)]
    with kept_team(32_000, lanes):
        for i, qlds in enumerate([1, 2, 2, 1, 2]):
            g = gs[i % 2]
            rc, dist, st = hm_sssp(g, i, d=d, qlds=qlds, rule=1, kfix=20, check_live=True, lanes=lanes)
            assert rc == 0 and st["first_bad"] == -1 and np.array_equal(dist, oracle.dijkstra(g, i)), (i, qlds)


@pytest.mark.parametrize("lanes", [0] + LANES)
@pytest.mark.parametrize("d", [1, 4])
def test_a_level_that_does_not_fit_is_reported(lanes, d):
    """B_1 and S_1 merge into a buffer of 16 d elements.  More than that breaks
    the heap's invariants: E_INTERNAL (-6), and nothing past the buffer is
    written.  (The form of one wavefront took it and wrote on.)"""
    for nB, nS in [(16 * d, 0), (12 * d, 4 * d), (16 * d - 1, 1), (8 * d, 8 * d)]:
        assert fill(d, nB, nS, lanes) == (0, False), (nB, nS)
    for nB, nS in [(16 * d, 1), (14 * d, 6 * d), (16 * d, 8 * d)]:
        assert fill(d, nB, nS, lanes) == (-6, False), (nB, nS)


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("seed", range(1, 5))
def test_the_order_of_the_lanes_does_not_show(lanes, seed):
    """Between the operations that all lanes (of a wavefront, of the team) take
    part in, they may run in any order: no lane reads what another writes in
    the same stretch."""
    with lane_order(seed, lanes):
        both(W.grid4(8, 9, 1, 100, 2), 0, lanes, qlds=2 * (seed % 2))
        both(W.random_graph(60, 900, 0, 5, 3), 0, lanes, qlds=1)
        both(W.random_graph(400, 4000, 0, 50, 3), 0, lanes, rule=1, kfix=100, kmax=256, d=40, qlds=seed % 2)
        with kept_team(60_000, lanes):
            rc, dist, st = hm_sssp(W.grid8(12, 12, 10000, 4), 0, rule=3, kseq=[7, 1, 40], kmax=256, d=32, qlds=1,
                                   lanes=lanes, check_live=True)
        assert rc == 0 and st["first_bad"] == -1
        assert np.array_equal(dist, oracle.dijkstra(W.grid8(12, 12, 10000, 4), 0))
        h, o = HostHeap(300, 7, 0, lanes), oracle.PQ(300)
        for op in W.random_script(12, 300, 60, 50, seed, deletes=True):
            a, b = getattr(h, {"update": "bulk_update", "extract": "extract_min"}.get(op[0], op[0])), \
                getattr(o, {"update": "bulk_update", "extract": "extract_min"}.get(op[0], op[0]))
            x, y = a(*op[1:]), b(*op[1:])
            if op[0] == "extract":
                assert all(np.array_equal(p, q) for p, q in zip(x, y))
