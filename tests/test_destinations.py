"""Which origin-destination pairs a handle accepts."""
import time

import numpy as np
import pytest

from paper_2603_25068_amd import workloads as W
from paper_2603_25068_amd.sim import SimError, footprint, lib


@pytest.mark.parametrize("turn_back", [False, True])
def test_destinations_across_components(turn_back):
    """Two two-way roads joined by a one-way link: agents may cross it one way only, and the first agent (whose
    component is looked at first) may be in either part."""
    w = W.line(n_links=5, n_agents=4)
    net = w.net
    net.n_nodes = 4
    net.tail[:], net.head[:] = [0, 1, 1, 2, 3], [1, 0, 2, 3, 2]   # 0 <-> 1 -> 2 <-> 3
    net.origin_node = np.asarray([0, 3, 1], np.int32)
    for first in (0, 1):
        w.dem.agent_origin[:] = [first, 0, 2, 1]
        w.dem.agent_dest[:] = [1 if first == 0 else 2, 3, 2, 0 if turn_back else 2]
        if turn_back:
            with pytest.raises(SimError, match="rejected"):
                footprint(w)
        else:
            assert footprint(w) > 0


def _lattice_with_inflows(n, n_dest, first_inflow):
    """An n x n lattice of two-way roads with a one-way inflow link to a corner, the origin of the first agent or of
    the second; destinations spread over the lattice."""
    roads = W.grid_roads(n, n)
    tail = np.concatenate([roads[:, 0], roads[:, 1], [n * n]])
    head = np.concatenate([roads[:, 1], roads[:, 0], [0]])
    w = W.line(n_links=len(tail), n_agents=n_dest)
    net = w.net
    net.n_nodes = n * n + 1
    net.tail[:], net.head[:] = tail, head
    net.origin_node = np.asarray([n * n, 0] if first_inflow else [0, n * n], np.int32)
    w.dem.agent_origin[:] = np.arange(n_dest) % 2
    w.dem.agent_dest[:] = 1 + np.arange(n_dest) % (n * n - 1)
    return w


def test_an_inflow_node_first_costs_no_search_per_destination():
    """The first agent's origin has no in-link, as virtual inflow nodes have none: 0.6 s for a search per destination
    against 0.02 s."""
    t = {}
    for first_inflow in (False, True):
        w = _lattice_with_inflows(64, 4000, first_inflow)
        best = np.inf
        for _ in range(3):
            t0 = time.perf_counter()
            assert footprint(w) > 0
            best = min(best, time.perf_counter() - t0)
        t[first_inflow] = best
    assert t[True] < 4 * t[False] + 0.05, t


@pytest.mark.parametrize("bad", [(), (7,), (3, 90), (90, 250, 299)])
def test_unreachable_destinations_among_one_way_roads(bad):
    """One-way corridors without any loop: every destination takes its own search; an agent placed downstream of its
    destination is found wherever it stands."""
    w = W.line(n_links=60, n_agents=300)
    rng = np.random.default_rng(len(bad))
    w.net.origin_node = np.arange(60).astype(np.int32)
    w.dem.agent_origin[:] = rng.integers(0, 59, 300)
    w.dem.agent_dest[:] = [rng.integers(o + 1, 61) for o in w.dem.agent_origin]
    for i in bad:
        w.dem.agent_origin[i], w.dem.agent_dest[i] = 40, 39
    if bad:
        with pytest.raises(SimError, match="rejected"):
            footprint(w)
        assert lib().sim_last_error(None).decode().startswith(f"agent {bad[0]}:")
    else:
        assert footprint(w) > 0
