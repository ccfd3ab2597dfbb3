"""The forms that the round loop picks by size and placement give one result:
levels in LDS (one wavefront in registers, lists sorted in LDS) against every
level in HBM (the general forms), and Select at the edges of its forms."""
import numpy as np
import pytest

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
    for n in (1, 3, nt - 1, nt + 1, 4 * nt, 4 * nt + 1, 16 * nt, 16 * nt + 1):
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
