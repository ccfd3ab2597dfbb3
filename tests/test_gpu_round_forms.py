"""The forms that the round loop picks by size and placement give one result:
levels in LDS (one wavefront in registers, lists sorted in LDS) against every
level in HBM (the general forms), and Select at the edges of its forms."""
import numpy as np
import pytest

import oracle
import paper_1908_09378_amd as pkg
import workloads as W
from gpu_util import dev32, run_sssp

pytestmark = pytest.mark.gpu
NO_LDS = 0xFFFFFFFF
GRAPHS = [W.grid4(31, 17, 1, 100, 3), W.grid4(9, 64, 0, 3, 4), W.grid8(23, 29, 10000, 5), W.ring_lattice(700, 16, 1, 1000, 6),
          W.random_graph(300, 3000, 0, 5, 7), W.random_graph(900, 5000, 0, 10 ** 6, 8), W.path_graph(80),
          W.random_graph(64, 2500, 1, 1 << 31, 9)]
SAME = ("rounds", "relaxations", "updates", "extracted", "heap_elems", "resolves")


def both(g, **kw):
    da, a = run_sssp(pkg, g, 0, **kw)
    db, b = run_sssp(pkg, g, 0, lds_levels=NO_LDS, **kw)
    assert np.array_equal(da, db)
    for s in SAME:
        assert a[s] == b[s], s


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("mult", [1, 2, 5])
def test_plain_rounds(gi, mult):
    g = GRAPHS[gi]
    both(g, d=mult * g.max_degree(), team=64)


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("team", [64, 256])
@pytest.mark.parametrize("k", [2, 37, 256])
def test_speculative_rounds(gi, team, k):
    g = GRAPHS[gi]
    kseq = dev32(np.array([k, 1, 3 * k, k // 2 + 1], np.uint32))
    both(g, d=max(64, g.max_degree()), team=team, k_rule=pkg.K_SEQ, k_seq=kseq, k_max=256)


@pytest.mark.parametrize("nt", [64, 256, 1024])
@pytest.mark.parametrize("spread", [1, 2, 200, 1 << 20, 1 << 63])
def test_select_edges(nt, spread):
    rng = np.random.default_rng(nt + spread % 1000)
    for n in (1, 3, nt - 1, nt + 1, 4 * nt, 4 * nt + 1, 16 * nt, 16 * nt + 1, 32 * nt, 32 * nt + 1):
        ids = rng.permutation(4 * n)[:n].astype(np.uint32)
        keys = rng.integers(0, spread, n, dtype=np.uint64) + np.uint64(7)
        order = np.lexsort((ids, keys))
        for r in sorted({1, 2, 3, n // 2, n - 3, n - 1, n} & set(range(1, n + 1))):
            res = run_select(nt, keys, ids, r)
            assert res == (int(keys[order[r - 1]]), int(ids[order[r - 1]])), (n, r)


def run_select(nt, keys, ids, r):
    import torch
    import devprims
    from gpu_util import dev64, host64
    ak, av = dev64(keys), dev32(ids)
    out = torch.zeros(8, dtype=torch.int64, device="cuda")
    rc = devprims.lib().dp_run(nt, 4, ak.data_ptr(), av.data_ptr(), len(ids), None, None, r, None, None, None, None,
                               None, None, None, out.data_ptr())
    assert rc == 0
    h = host64(out)
    return int(h[0]), int(h[1])


def skewed(n, hub, deg, seed):
    """`deg` edges from each vertex, one after another on a ring, some without
    any, and two hubs of `hub` edges."""
    rng = np.random.default_rng(seed)
    cnt = np.full(n, deg, np.int64)
    cnt[rng.integers(1, n, n // 8)] = 0
    cnt[[0, n // 2]] = hub
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.uint64)
    m = int(off[-1])
    src = np.repeat(np.arange(n), cnt)
    tg = ((src + rng.integers(1, 3 * deg + 2, m)) % n).astype(np.uint32)
    far = rng.random(m) < 0.2
    tg[far] = rng.integers(0, n, int(far.sum()))
    return W.csr_from_edges(n, src, tg, rng.integers(0, 50, m).astype(np.uint32), "skewed")


@pytest.mark.parametrize("team", [64, 256, 1024])
@pytest.mark.parametrize("hub,deg", [(0, 1), (5, 4), (64, 16), (700, 3), (2100, 24), (9000, 2)])
def test_whose_edge_is_whose(team, hub, deg):
    """The two ways of dealing out the edges of a round (groups of lanes for
    even degrees, a search for others), with one and with several passes."""
    g = skewed(997, hub or 1, deg, hub + deg)
    ref = oracle.dijkstra(g, 0)
    for k in (1, 2, 63, 64, 256):
        d, _ = run_sssp(pkg, g, 0, d=max(64, g.max_degree()), team=team, k_rule=pkg.K_FIXED, k_fixed=k, k_max=256)
        assert np.array_equal(d, ref), k


@pytest.mark.parametrize("nq", [3, 600])
def test_batch_lists(nq):
    """Round lists in LDS (few queries) and as far as residency leaves room."""
    import torch
    from gpu_util import DEV, graph_to_dev, host64
    gs = [W.grid4(31, 17, 1, 100, 3), skewed(600, 200, 5, 1), W.path_graph(80)]
    dg = [graph_to_dev(g) for g in gs]
    qs, refs = [], []
    for i in range(nq):
        g = gs[i % 3]
        s = i % 7
        qs.append((*dg[i % 3], g.n, g.m, s, torch.empty(g.n, dtype=torch.int64, device=DEV)))
        refs.append(oracle.dijkstra(g, s))
    for team in (64, 256):
        for q in qs:
            q[6].fill_(7)
        pkg.sssp_batch(qs, k_rule=pkg.K_FIXED, k_fixed=40, k_max=256, team=team)
        for q, ref in zip(qs, refs):
            assert np.array_equal(host64(q[6]), ref)


@pytest.mark.parametrize("team,scale", [(64, 18), (256, 15)])
def test_batch_teams_go_from_staged_queries_to_others(team, scale):
    """More queries than resident teams, the larger ones with a staging area
    after their LDS levels (8 edges a vertex: one level of d = 144 or 120) and
    the others, taken by the same teams later, with LDS levels in its place (4
    edges: two levels of d = 72 or 60) and merges in HBM that are large enough
    for one."""
    import torch
    from gpu_util import DEV, graph_to_dev, host64
    n, each = 6000, 700
    rng = np.random.default_rng(team)
    qs, refs = [], []
    for deg in (8, 4):
        g = W.csr_from_edges(n, np.repeat(np.arange(n), deg), rng.integers(0, n, n * deg),
                             rng.integers(0, 10 ** 6, n * deg).astype(np.uint32), f"out{deg}")
        assert g.max_degree() == deg
        dg = graph_to_dev(g)
        ref = [oracle.dijkstra(g, s) for s in range(5)]
        for i in range(each):
            qs.append((*dg, n, g.m, i % 5, torch.empty(n, dtype=torch.int64, device=DEV)))
            refs.append(ref[i % 5])
    pkg.sssp_batch(qs, d_scale=scale, team=team, k_rule=pkg.K_FIXED, k_fixed=64, k_max=256)
    for q, ref in zip(qs, refs):
        assert np.array_equal(host64(q[6]), ref)


@pytest.mark.parametrize("team", [256, 1024])
@pytest.mark.parametrize("d", [101, 520, 1100, 4097])
def test_staged_merges(team, d):
    """Merges of HBM levels below, at and above whole and half tiles of the
    staging area, and Select over up to 32 elements per thread."""
    g = W.random_graph(4000, 90000, 0, 10 ** 6, d)
    ref = oracle.dijkstra(g, 0)
    dist, _ = run_sssp(pkg, g, 0, d=d, team=team, lds_levels=NO_LDS)
    assert np.array_equal(dist, ref)
    kseq = dev32(np.array([90, 1, 200, 7], np.uint32))
    dist, _ = run_sssp(pkg, g, 0, d=d, team=team, lds_levels=NO_LDS, k_rule=pkg.K_SEQ, k_seq=kseq, k_max=256)
    assert np.array_equal(dist, ref)


@pytest.mark.parametrize("d", [100, 101, 159, 163, 167, 256, 257])
def test_team_by_bulk_size(d):
    g = W.ring_lattice(900, 30, 1, 1000, 3)
    dist, st = run_sssp(pkg, g, 0, d=d)
    assert np.array_equal(dist, oracle.dijkstra(g, 0))
    _, one = run_sssp(pkg, g, 0, d=d, team=64)
    assert st["lds_levels"] == one["lds_levels"] or d > 256
    for s in SAME[:4]:
        assert st[s] == one[s], s
