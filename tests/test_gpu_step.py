"""The fused step where its paths meet: one workgroup for a whole network, one launch per step over every
mixture of node and link classes; rollouts cut at any point, which moves the state between the live copies
and the tape; agents placed out of position order; captured steps.  Everything forward is exact (the oracle's
positions are float with the same operations; integers are integers); gradients of the same rollout cut
differently are bitwise the same."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2603_25068_amd import workloads as W
from test_gpu_parity import _compare_state, _grad_close, _sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,lanes,S", [(2, 2, 1, 1), (6, 6, 2, 1), (6, 6, 2, 3), (7, 7, 3, 1), (9, 5, 8, 1),
                                           (16, 16, 3, 2), (10, 10, 2, 60)])
def test_step_paths_against_the_oracle(nx, ny, lanes, S):
    w = W.random_small(nx + ny, nx=nx, ny=ny, n_agents=20 * nx * ny, rates=True, steps=160, lanes_max=lanes)
    seeds = [100 + k for k in range(S)]
    s = _sim(w, n_scenarios=S, seeds=seeds)
    s.step(97)
    s.step(1)
    s.step(62)
    for k in {0, S // 2, S - 1}:
        o = Oracle(w, seed=seeds[k]).run()
        _compare_state(o, s, scen=k, ctx=f"scenario {k}")
        assert np.array_equal(o.counts()[0].astype(np.float32), s.observables()[0][k])


@pytest.mark.parametrize("spokes,lanes,sched", [(3, 1, (8, 8, 8)), (8, 8, (64, 64, 8)), (8, 8, (8, 64, 8)), (5, 3, (16, 32, 8)),
                                                (12, 5, (32, 64, 8)), (40, 1, (8, 64, 8))])
def test_step_classes_against_the_oracle(spokes, lanes, sched):
    """Node and link classes with fewer tasks than a row of workgroups, with several, and with none; four
    scenarios a launch."""
    w = W.hub(n_spokes=spokes, lanes=lanes, n_agents=1200, steps=160, seed=spokes)
    seeds = [7, 8, 9, 10]
    s = _sim(w, n_scenarios=4, seeds=seeds)
    s.set_schedule(*sched)
    s.rollout()
    for k in range(4):
        o = Oracle(w, seed=seeds[k]).run()
        _compare_state(o, s, scen=k, ctx=f"scenario {k}")
        assert np.array_equal(o.counts()[0].astype(np.float32), s.observables()[0][k])


@pytest.mark.parametrize("nx", [4, 9])
@pytest.mark.parametrize("cuts", [(160,), (1,) * 7 + (153,), (33, 3, 24, 40, 60), (40, 40, 40, 39, 1)])
def test_cut_rollouts_leave_the_same_state_and_tape(nx, cuts):
    """Windows of 40 steps: calls that end inside, at and one step from a window's end."""
    w = W.random_small(5, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=160, lanes_max=3)
    whole = _sim(w, record=True, ckpt_every=40).rollout()
    cut = _sim(w, record=True, ckpt_every=40)
    for n in cuts:
        cut.step(n)
    a, b = whole.state(), cut.state()
    for k in ("status", "link", "pos", "seq"):
        assert np.array_equal(a[k], b[k]), k
    gQ = np.random.default_rng(nx).normal(size=whole.observables()[0].shape).astype(np.float32)
    gx = np.random.default_rng(nx + 1).normal(size=(1, w.dem.n_agents)).astype(np.float32)
    groups = ("free_speed", "jam_density", "rates", "cap_mult", "beta", "alpha")
    for gs in (groups[:3], groups):
        ga, gb = whole.backward(gQ=gQ, gT=[0.2], gx=gx, groups=gs), cut.backward(gQ=gQ, gT=[0.2], gx=gx, groups=gs)
        for k in gs:
            assert np.array_equal(ga[k], gb[k]), k
    o = Oracle(w, log=True).run()
    go = o.backward(gQ=gQ[0].astype(np.float64), gT=0.2, gx=gx[0].astype(np.float64))
    for k in groups:
        _grad_close(go[k], gb[k][0], k)


def test_placement_out_of_position_order():
    """A caller may place agents on a link back to front.  Entry slots then count the whole ring: the agent
    placed first creeps from 1 m at 1 m/s and keeps the one-lane entry (5 m) taken until its fifth step,
    although the agent behind it in the ring stands at 100 m; also after the state went through a blob."""
    w = W.line(n_links=2, length=200.0, speed=1.0, n_agents=3, ready=np.zeros(3), steps=12)
    s, q = _sim(w), _sim(w)
    s.place([0, 1], [0, 0], [1.0, 100.0])
    q.set_full_state(s.full_state())
    for x in (s, q):
        for t in range(8):
            x.step()
            st = x.state()
            assert st["status"][0][2] == (2 if t >= 4 else 1), t
            assert st["pos"][0][0] == 2.0 + t and st["pos"][0][1] == 100.0, t
            assert st["counters"][0]["order_viol"] == t + 1


@pytest.mark.parametrize("head,tail", [(5, 4), (0, -1), (-1, 3), (-2, -2)])
def test_state_blobs_with_bad_ring_counters_are_refused(head, tail):
    """A ring's free slots follow from its head and length: a blob whose counters do not belong together is
    refused before it changes anything."""
    import struct
    from paper_2603_25068_amd.sim import SimError
    w = W.random_small(12, nx=4, ny=4, n_agents=300, rates=True, steps=120)
    s = _sim(w)
    s.step(40)
    blob = s.full_state()
    slots = struct.unpack_from("<q", blob, 56)[0]
    links = 64 + slots * (4 + 4 + 8)            # positions, agents, destinations; then 32 bytes a link
    bad = bytearray(blob)
    struct.pack_into("<ii", bad, links + 32 * (w.net.n_links - 1) + 16, head, tail)
    s.step(3)
    before = s.full_state()
    with pytest.raises(SimError, match="ring counters"):
        s.set_full_state(bytes(bad))
    assert s.full_state() == before
    s.step(5)
    _compare_state(Oracle(w).run(48), s)


@pytest.mark.parametrize("nx,n", [(4, 3), (9, 3), (9, 4)])
def test_captured_steps_replay(nx, n):
    """n captured steps (odd and even) replayed with eager work between: each replay equals an eager run of
    the same steps from the state before it."""
    import struct
    import torch
    w = W.random_small(6, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st), _sim(w)
    s.step(50)
    e.step(50)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        s.step(n)
    for k in range(4):
        with torch.cuda.stream(st):
            g.replay()
            torch.zeros(1000, device="cuda").sum()
        st.synchronize()
        e.step(n)
        a, b = s.state(), e.state()
        for key in ("status", "link", "pos", "seq"):
            assert np.array_equal(a[key], b[key]), (k, key)
        blob = bytearray(e.full_state())                       # the eager run goes back to step 50, as a replay does
        assert struct.unpack_from("<i", blob, 36)[0] == 50 + n
        struct.pack_into("<i", blob, 36, 50)
        e.set_full_state(bytes(blob))


@pytest.mark.parametrize("S", [1, 3])
def test_tapes_follow_the_groups_of_the_last_backward(S):
    """The forward tapes capacity and straight-through factors once a backward has asked for them.  The first
    pass replays every window, the second sweeps the forward's tapes, the third asks for less, the fourth for
    another subset again: every gradient bitwise as in the first pass."""
    w = W.random_small(21, nx=5, ny=5, n_agents=700, rates=True, steps=200, lanes_max=3)
    s = _sim(w, n_scenarios=S, record=True, ckpt_every=40)
    every = ("free_speed", "jam_density", "rates", "cap_mult", "beta", "cost", "alpha", "theta")
    ref = None
    for groups in (every, every, ("free_speed", "cap_mult"), every[:3], ("beta", "cap_mult"), every):
        s.reset()
        s.rollout()
        cnt, _ = s.observables()
        gQ = np.random.default_rng(3).normal(size=cnt.shape).astype(np.float32)
        g = s.backward(gQ=gQ, gT=[0.4] * S, groups=groups)
        ref = ref or g
        for k in groups:
            assert np.array_equal(g[k], ref[k]), (groups, k)


@pytest.mark.parametrize("agents,S", [(1, 1), (13, 3), (16, 2), (37, 1)])
def test_reset_clears_every_array_to_its_last_byte(agents, S):
    """Agent arrays of 1 to 39 bytes a scenario: whole 16-byte chunks, tails, and tails alone."""
    w = W.random_small(agents, nx=3, ny=3, n_agents=agents, steps=60)
    w.dem.ready_time[:] = 0
    seeds = [3 + k for k in range(S)]
    s = _sim(w, n_scenarios=S, seeds=seeds, record=True)
    gQ = np.ones((S,) + s.observables()[0].shape[1:], np.float32)
    first = None
    for _ in range(3):
        s.reset()
        st = s.state()
        assert not st["status"].any() and (st["link"] < 0).all()
        s.rollout()
        for k in range(S):
            _compare_state(Oracle(w, seed=seeds[k]).run(), s, scen=k)
        g = s.backward(gQ=gQ, gT=[1.0] * S, groups=("free_speed", "beta", "cost"))
        first = first or g
        for k in g:
            assert np.array_equal(first[k], g[k]), k
