"""The straight-through kernel at hubs of many shapes against the oracle: out-degrees on both sides of
its register blocks (4, 8 and above), lane groups of 8 to 64 candidates, several winners per merge, a
small and a large temperature.  Tolerance: the adjoint is carried in float on the GPU, so a gradient
summed over steps agrees with the oracle's double one to the repository's 1e-3."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2603_25068_amd import workloads as W
from test_gpu_parity import _compare_state, _grad_close, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spokes,lanes,tau", [(2, 3, 0.5), (4, 2, 0.5), (5, 8, 0.5), (8, 8, 0.1), (9, 7, 0.5),
                                              (12, 5, 2.0), (20, 3, 0.5), (33, 1, 0.5)])
def test_straight_through_hub_shapes(spokes, lanes, tau):
    w = W.hub(n_spokes=spokes, lanes=lanes, n_agents=1500, steps=200, seed=spokes)
    w.cfg.gumbel_tau = tau
    w.cfg.ckpt_every = 60
    groups = ("beta", "cost", "alpha", "theta")
    s = _sim(w, record=True).rollout()
    o = Oracle(w, log=True).run()
    _compare_state(o, s)
    cnt, _ = s.observables()
    gQ = np.random.default_rng(spokes).normal(size=cnt.shape).astype(np.float32)
    gg = s.backward(gQ=gQ, gT=np.array([0.3]), groups=groups)
    go = o.backward(gQ=gQ[0].astype(np.float64), gT=0.3)
    for g in groups:
        _grad_close(go[g], gg[g][0], g)
