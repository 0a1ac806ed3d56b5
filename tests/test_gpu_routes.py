"""Route choice on the route table against the oracle, whose shortest times are Dijkstra's: networks around a
workgroup's 1024 threads, corridors (as many rounds as links; nodes that cannot reach the destination), one above
the LDS limit of 19,800 nodes, and chains that the kernel gives up.  Exact: the same doubles give the same choices."""
import time

import numpy as np
import pytest

from oracle import Oracle
from paper_2603_25068_amd import workloads as W
from test_gpu_parity import _compare_state, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,agents", [(1, 2, 8), (33, 31, 400), (32, 32, 400), (41, 25, 400), (140, 141, 30),
                                          (143, 141, 30)])
def test_lattice_routes(nx, ny, agents):
    w = W.random_small(nx, nx=nx, ny=ny, n_agents=agents, steps=80)
    w.cfg.dest_logit_coef = 0.2
    s = _sim(w).rollout()
    o = Oracle(w).run()
    _compare_state(o, s)
    assert o.counters()["departed"] > 0


def test_corridor_routes():
    w = W.line(n_links=1500, length=20.0, n_agents=20, steps=80)
    s = _sim(w).rollout()
    _compare_state(Oracle(w).run(), s)
    assert np.array_equal(s.dist_table(), Oracle(w).dist_table())


def _two_way_chain(n, n_dest, n_agents=None, speed=13.9, shortcut=None):
    """A two-way road of n nodes, destinations spread along it; with `shortcut` a slow two-way link from every
    `shortcut`-th node to one more node."""
    a = np.arange(n - 1)
    tail, head = np.concatenate([a, a + 1]), np.concatenate([a + 1, a])
    u = np.full(2 * n - 2, speed)
    if shortcut:
        k = np.arange(0, n, shortcut)
        tail, head = np.concatenate([tail, k, np.full(len(k), n)]), np.concatenate([head, np.full(len(k), n), k])
        u = np.concatenate([u, np.full(2 * len(k), 1e-4)])
    N = n_agents or max(n_dest, 10)
    w = W.line(n_links=len(tail), length=40.0, n_agents=N, steps=40)
    net = w.net
    net.n_nodes = n + bool(shortcut)
    net.tail[:], net.head[:], net.free_speed[:] = tail, head, u
    net.origin_node = np.asarray([0, n // 3, n - 1], np.int32)
    w.dem.agent_origin[:] = np.arange(N) % 3
    dest = np.resize(np.linspace(1, n - 3, n_dest).astype(np.int32), N)
    w.dem.agent_dest[:] = dest + (dest == net.origin_node[w.dem.agent_origin])
    w.dem.ready_time[:] = np.arange(N) % 20
    w.cfg.dest_logit_coef = 0.5
    return w


@pytest.mark.parametrize("n,n_dest,shortcut", [(300, 200, None), (1500, 40, None), (6000, 64, 100), (6000, 64, 200)])
def test_chain_routes(n, n_dest, shortcut):
    """Device by length and number of destinations, host, and chains of fast links whose slow shortcuts make them look
    short, so that the kernel starts and gives up."""
    w = _two_way_chain(n, n_dest, shortcut=shortcut)
    s = _sim(w).rollout()
    o = Oracle(w).run()
    _compare_state(o, s)
    assert o.counters()["transfers"] > 0
    assert np.array_equal(s.dist_table(), o.dist_table())


def test_creation_of_deep_networks():
    """A chain just inside the nodes that fit the kernel and one just outside, which takes the host's way: a launch per
    hop took ten times as long."""
    ms = {}
    for n in (19_700, 20_100):
        w, best = _two_way_chain(n, 8), np.inf
        for _ in range(3):
            t = time.perf_counter()
            _sim(w).close()
            best = min(best, time.perf_counter() - t)
        ms[n] = best * 1e3
    assert ms[19_700] < 3 * ms[20_100], ms
