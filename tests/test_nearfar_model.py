"""Near-Far's phases and grid barrier on the CPU (tests/hostmodel/
nearfar_model.hip): the kernel's code on workgroups of 4 threads, interleaved
at every access to shared memory."""
import numpy as np
import pytest

import oracle
import workloads as W
import hostmodel as hm

# light and heavy vertices (more than 6 out-edges), frontiers of one and of
# several workgroups, more pushes than a workgroup gathers (8)
GRAPHS = [W.grid4(6, 6, 1, 5, 3), W.random_graph(40, 160, 0, 9, 3), W.random_graph(60, 600, 1, 20, 4), W.path_graph(12)]


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("workgroups", [1, 3, 10])
@pytest.mark.parametrize("glog", [0, 1])
@pytest.mark.parametrize("delta", [1, 4, 1 << 40])
def test_threads_in_turn(gi, workgroups, glog, delta):
    g = GRAPHS[gi]
    rc, dist = hm.nearfar(g, 0, delta, glog, workgroups)
    assert rc == 0 and np.array_equal(dist, oracle.dijkstra(g, 0))


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("workgroups", [2, 3, 10])
def test_a_late_thread_stays_in_step(gi, workgroups):
    """Any thread may be late at any point: the threads of a workgroup still
    meet at the same barriers, and the run ends with the right distances.
    (Thread 0 of the barrier's leader once wrote the flag again that the
    others had yet to read.)"""
    g = GRAPHS[gi]
    ref = oracle.dijkstra(g, 0)
    for seed in range(60):
        rc, dist = hm.nearfar(g, 0, 4, 0, workgroups, hm.PRIORITY, seed=seed)
        assert rc == 0 and np.array_equal(dist, ref), seed


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("workgroups", [9, 10, 17])
def test_stores_may_land_late(gi, workgroups):
    """A store may reach the other workgroups at any time until its thread
    waits for its own operations.  (The reset of a group's arrivals was not
    waited for: with several workgroups to a group, it could undo an arrival
    at the next barrier.)"""
    g = GRAPHS[gi]
    ref = oracle.dijkstra(g, 0)
    for seed in range(150):
        rc, dist = hm.nearfar(g, 0, 4, 0, workgroups, hm.PRIORITY, True, seed)
        assert rc == 0 and np.array_equal(dist, ref), seed


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("workgroups", [2, 9])
def test_a_group_of_lanes_scans_at_one_distance(gi, workgroups):
    """The lanes that share a vertex agree on its distance, also when it falls
    while they read it.  (Each decided by its own read: the mark could name a
    smaller distance than the one that a lane relaxed its edges with.)"""
    g = GRAPHS[gi]
    ref = oracle.dijkstra(g, 0)
    for seed in range(60):
        rc, dist = hm.nearfar(g, 0, 4, 1, workgroups, hm.PRIORITY, bool(seed & 1), seed)
        assert rc == 0 and np.array_equal(dist, ref), seed
