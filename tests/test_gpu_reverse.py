"""The reverse kernel against the oracle on rings from a few ranks to several batches of rounds: 1 to 8
lanes (the leader's lane in the same round or the one before, up to a whole round of 8), 8 to 64 lanes a
link, cotangents of counts, travel time and final positions, with and without the straight-through blocks
in its launches, tape windows that the rollout leaves part-filled.  Tolerance: the adjoint is carried in
float on the GPU, so a gradient summed over steps agrees with the oracle's double one to the repository's
1e-3."""
import numpy as np
import pytest

import oracle
from oracle import Oracle
from paper_2603_25068_amd import workloads as W
from test_gpu_parity import _compare_state, _grad_close, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes,per_link,ste", [(1, 8, False), (2, 8, True), (3, 16, False), (5, 8, False),
                                                (7, 32, True), (8, 8, True), (8, 16, False), (8, 64, False)])
def test_reverse_ring_shapes(lanes, per_link, ste):
    w = W.hub(n_spokes=4, lanes=lanes, n_agents=1500, steps=232, seed=lanes)
    s = _sim(w, record=True, ckpt_every=60)
    s.set_schedule(8, s.schedule()[1], per_link)
    s.rollout()
    o = Oracle(w, log=True).run()
    _compare_state(o, s)
    st = o.state()
    on = st["status"] == oracle.ST_ON
    if lanes == 8:   # more than a batch of rounds on one link, whatever the lane group
        assert np.bincount(st["link"][on]).max() > 4 * 64
    rng = np.random.default_rng(lanes)
    cnt, _ = o.counts()
    gQ = rng.normal(size=cnt.shape).astype(np.float32)
    gx = (rng.normal(size=w.dem.n_agents) * on).astype(np.float32)
    groups = ("free_speed", "jam_density", "rates") + (("beta", "cost") if ste else ("cap_mult",))
    go = o.backward(gQ=gQ.astype(np.float64), gT=0.3, gx=gx.astype(np.float64))
    gg = s.backward(gQ=gQ[None], gT=[0.3], gx=gx[None], groups=groups)
    for g in groups:
        _grad_close(go[g], gg[g][0], g)
