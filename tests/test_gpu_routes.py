"""Route choice on the device's route table against the oracle, whose shortest times are Dijkstra's: networks
around a workgroup's 1024 threads, a corridor of 1,500 links (as many rounds as links; nodes that cannot reach
the destination), and one above the LDS limit of 19,800 nodes.  Exact: the same doubles give the same choices."""
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
