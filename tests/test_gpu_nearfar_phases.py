"""Near-Far phases at the edges of their forms: frontiers of one workgroup and
just above, more pushes per workgroup than its gather holds, far piles."""
import numpy as np
import pytest

import oracle
import paper_1908_09378_amd as pkg
import workloads as W
from gpu_util import DEV, graph_to_dev, host64

pytestmark = pytest.mark.gpu


def layers(width, depth, seed):
    """`depth` layers of `width` vertices, each linked to three of the next
    layer: every frontier has about `width` vertices."""
    rng = np.random.default_rng(seed)
    n = 1 + width * depth
    src, dst = [np.zeros(width, np.int64)], [np.arange(1, width + 1)]
    for l in range(depth - 1):
        v = 1 + l * width + np.arange(width)
        for s in range(3):
            src.append(v)
            dst.append(1 + (l + 1) * width + (np.arange(width) + s) % width)
    src, dst = np.concatenate(src), np.concatenate(dst)
    return W.csr_from_edges(n, src, dst, rng.integers(1, 4, src.size), f"layers_{width}x{depth}")


def check(g, delta):
    import torch
    off, tg, wt = graph_to_dev(g)
    dist = torch.empty(g.n, dtype=torch.int64, device=DEV)
    pkg.sssp_nearfar(off, tg, wt, g.n, g.m, 0, dist, delta)
    assert np.array_equal(host64(dist), oracle.dijkstra(g, 0))


@pytest.mark.parametrize("width", [1, 127, 128, 129, 513, 2000])
@pytest.mark.parametrize("delta", [0, 1, 5])
def test_frontier_widths(width, delta):
    check(layers(width, 12, width), delta)


@pytest.mark.parametrize("delta", [0, 1, 700, 1 << 40])
def test_more_pushes_than_a_workgroup_gathers(delta):
    # degrees of about 1,000, below the threshold of the whole-grid scan:
    # eight vertices of a workgroup push up to 8,000 targets in one phase
    g = W.random_graph(20000, 600_000, 1, 1000, 3)
    check(g, delta)
    rng = np.random.default_rng(5)
    hubs, leaves = 64, 40000
    src = np.concatenate([np.zeros(hubs, np.int64), np.repeat(1 + np.arange(hubs), 1000)])
    dst = np.concatenate([1 + np.arange(hubs), 1 + hubs + rng.integers(0, leaves, hubs * 1000)])
    check(W.csr_from_edges(1 + hubs + leaves, src, dst, rng.integers(1, 2000, src.size), "hubs"), delta)
