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


def _fifo_roads(n_links, place, T, lanes, length, u, kappa, n_queued):
    """One-link roads as the library steps them, agents in placed order (the oracle ranks agents by position): each
    agent behind the one `lanes` ahead of it in the ring; as many heads leave as agents of the whole ring have
    arrived, at most `lanes`; the next of the road's waiting agents enters if an entry slot is free.  With each
    agent's derivatives to its road's speed and jam density, held branches as the adjoint has them (positions:
    float; derivatives: double)."""
    f = np.float32
    rings = [[] for _ in range(n_links)]
    for a, (j, x) in enumerate(place):
        rings[j].append([a, f(x), 0.0, 0.0])
    a = len(place)
    queue = [list(range(a + j * n_queued, a + (j + 1) * n_queued)) for j in range(n_links)]
    exited, viol, full = set(), 0, 0
    for _ in range(T):
        for j, ring in enumerate(rings):
            ln, sp = lanes[j], f(1.0) / f(kappa[j])
            viol += sum(p[1] < q[1] for p, q in zip(ring, ring[1:]))
            new = []
            for r, (a, x, su, sk) in enumerate(ring):
                xf, lead = f(x + f(u[j])), ring[r - ln] if r >= ln else None
                cc = max(x, f(lead[1] - sp)) if lead else None
                if lead is None or xf <= cc:
                    n = [a, xf, su + 1.0, sk]
                elif x > f(lead[1] - sp):
                    n = [a, x, su, sk]
                else:
                    n = [a, cc, lead[2], lead[3] + 1.0 / float(f(kappa[j])) ** 2]
                n[1] = min(n[1], f(length[j]))
                new.append(n)
            arrived = [n[1] >= f(length[j]) - f(0.01) for n in new]
            taken = [n[1] <= sp for n in new]
            h = min(sum(arrived), ln)
            full += (h != sum(arrived[:ln])) + (min(sum(taken), ln) != sum(taken[-ln:]))
            exited.update(n[0] for n in new[:h])
            new = new[h:]
            if sum(taken) < ln and queue[j]:
                new.append([queue[j].pop(0), f(0), 0.0, 0.0])
            rings[j] = new
    return rings, exited, viol, full


@pytest.mark.parametrize("n_links,T,per_lane", [(6, 45, 4), (260, 45, 4), (8, 30, 40), (60, 30, 40)])
def test_out_of_order_rings_step_and_reverse(n_links, T, per_lane):
    """Links of 1, 2, 3 and 8 lanes with agents placed in any order, some on the entry slots behind others, some at
    the end of their link behind others that are not: arrivals and entry slots of whole rings, and the gradients
    of such a run; networks in one workgroup and with a launch per step, also continued from a blob; short rings and
    rings of up to 340 agents."""
    rng = np.random.default_rng(n_links)
    lanes = np.resize([1, 2, 3, 8], n_links)
    length = rng.uniform(60.0, 300.0, n_links).astype(np.float32)
    u = rng.uniform(1.0, 14.0, n_links).astype(np.float32)
    kappa = rng.uniform(0.18, 0.22, n_links).astype(np.float32)
    place = []
    for j in range(n_links):
        k = int(rng.integers(0, min(per_lane * lanes[j] + 4, lanes[j] * length[j] / 7)))
        x = rng.uniform(0, length[j], k)
        x[rng.random(k) < 0.3] = length[j]
        near = rng.random(k) < 0.3
        x[near] = rng.uniform(0, 4.0, near.sum())
        place += [(j, np.float32(min(v, length[j]))) for v in x]
    n_queued, P = 5, len(place)
    N = P + n_queued * n_links
    w = W.line(n_links=n_links, n_agents=N, ready=np.zeros(N), steps=T)
    net = w.net
    net.n_nodes = 2 * n_links
    net.tail[:], net.head[:] = 2 * np.arange(n_links), 2 * np.arange(n_links) + 1
    net.lanes[:], net.length[:], net.free_speed[:], net.jam_density[:] = lanes, length, u, kappa
    net.detector_pos[:] = length * np.float32(0.5)
    net.origin_node = np.arange(0, 2 * n_links, 2).astype(np.int32)
    road = np.concatenate([[j for j, _ in place], np.repeat(np.arange(n_links), n_queued)]).astype(np.int32)
    w.dem.agent_origin[:], w.dem.agent_dest[:] = road, 2 * road + 1
    rings, exited, viol, full = _fifo_roads(n_links, place, T, lanes, length, u, kappa, n_queued)
    assert full > 5   # steps whose counts the ends of the ring alone would get wrong
    s = _sim(w, record=True, ckpt_every=10, tape_windows=4)
    s.place(np.arange(P), road[:P], [x for _, x in place])
    half = _sim(w)
    s.step(T // 2)
    half.set_full_state(s.full_state())
    half.step(T - T // 2)
    s.step(T - T // 2)
    for x in (s, half):
        st = x.state()
        assert set(np.flatnonzero(st["status"][0] == 3)) == exited
        assert st["counters"][0]["order_viol"] == viol
        for j, ring in enumerate(rings):
            on = np.flatnonzero(st["link"][0] == j)
            on = on[np.argsort(st["seq"][0][on])]
            assert on.tolist() == [n[0] for n in ring], j
            assert np.array_equal(st["pos"][0][on], np.array([n[1] for n in ring], np.float32)), j
    one = s.state()
    for S in (3, 8):   # a launch's workgroups in rows, and packed
        m = _sim(w, n_scenarios=S)
        m.place(np.arange(P), road[:P], [x for _, x in place])
        m.step(T)
        st = m.state()
        for key in ("status", "link", "pos", "seq"):
            assert (st[key] == one[key]).all(), (S, key)
    gx = rng.normal(size=(1, N)).astype(np.float32)
    g = s.backward(gx=gx, groups=("free_speed", "jam_density"))
    for k, name in ((2, "free_speed"), (3, "jam_density")):
        want = np.array([sum(float(gx[0, n[0]]) * n[k] for n in ring) for ring in rings])
        size = np.array([sum(abs(float(gx[0, n[0]]) * n[k]) for n in ring) for ring in rings])
        # float adjoints: a sum of at most T (N / links + 1) rounded terms, of the size of the absolute terms
        assert (np.abs(g[name][0] - want) <= 1e-5 * size + 1e-12).all(), name


@pytest.mark.parametrize("S", [256, 257, 600])
def test_many_scenarios_of_a_small_network(S):
    """One workgroup a scenario as long as all run at once, a launch per step beyond that."""
    w = W.random_small(14, nx=3, ny=3, n_agents=120, rates=True, steps=80, lanes_max=3)
    seeds = [50 + k for k in range(S)]
    s = _sim(w, n_scenarios=S, seeds=seeds, record=True, ckpt_every=30)
    s.rollout()
    st, ls = s.state(), s.link_state()
    for k in {0, 1, S // 2, 255, S - 1}:
        o = Oracle(w, seed=seeds[k]).run()
        so, lo = o.state(), o.link_state()
        on = so["status"] == 2
        for key in ("link", "pos", "seq"):
            assert np.array_equal(so[key][on].astype(np.float32), st[key][k][on].astype(np.float32)), (k, key)
        assert np.array_equal(so["status"], st["status"][k]), k
        for key in lo:
            assert np.array_equal(lo[key], ls[key][k]), (k, key)
    one = _sim(w, seeds=[seeds[-1]], record=True, ckpt_every=30).rollout()
    groups = ("free_speed", "cap_mult", "beta")
    g, h = s.backward(gT=[1.0] * S, groups=groups), one.backward(gT=[1.0], groups=groups)
    for k in groups:
        assert np.array_equal(g[k][-1], h[k][0]), k


def test_steps_of_many_scenarios_fill_the_chip():
    """Four times the scenarios that one workgroup each holds at once: not four times the step (3.9 times with a
    workgroup each, 1.3 with packed launches)."""
    import time
    import torch
    w = W.diamond(200)
    us = {}
    for S in (256, 1024):
        s, best = _sim(w, n_scenarios=S), np.inf
        for _ in range(5):
            s.reset()
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.step(200)
            best = min(best, time.perf_counter() - t)
        us[S] = best / 200 * 1e6
    assert us[1024] < 2.2 * us[256], us


def test_restored_placements_step_as_fast_as_placed_ones():
    """A blob whose placed agents stand in order: the steps after it take no full-ring counts (fifteen times the time
    on these rings of hundreds of agents; a factor of 1.6 allows for noise)."""
    w = W.hub(n_spokes=8, lanes=8, n_agents=12000, steps=300)
    net = w.net
    links, pos = [], []
    for j in range(net.n_links):
        k = np.arange(int(net.lanes[j] * net.length[j] * 0.1))
        links.append(np.full(len(k), j))
        pos.append(net.length[j] * (1 - (k // net.lanes[j] * net.lanes[j]) / (2.0 * len(k))))
    links, pos = np.concatenate(links), np.concatenate(pos)
    s = _sim(w)
    s.place(np.arange(len(links)), links, pos)
    blob = s.full_state()
    ms = {}
    for name in ("placed", "restored"):
        best = np.inf
        for _ in range(3):
            if name == "placed":
                s.reset()
                s.place(np.arange(len(links)), links, pos)
            else:
                s.set_full_state(blob)
            s.set_timing(True)
            s.step(60)
            best = min(best, s.timing()["link_ev"][0])
            s.set_timing(False)
        ms[name] = best
    assert ms["restored"] < 1.6 * ms["placed"], ms


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


def test_schedules_of_other_kernels_are_probed_again(tmp_path):
    """A cache file from kernels with another work split: its entries are read over, not applied; the file goes on
    being used."""
    w = W.random_small(16, nx=5, ny=5, n_agents=500, rates=True, steps=120)
    path = tmp_path / "schedules.txt"
    _sim(w, n_scenarios=5).autotune(probe_steps=4, cache_path=str(path))
    key = path.read_text().split()[0]
    assert "/k" in key
    old = key[:key.index("/k")].replace("/S5/", "/S6/")   # as a file from before the revision names six scenarios
    path.write_text(f"{old} 64 64 64 1.0\n")
    s = _sim(w, n_scenarios=6)
    sched = s.autotune(probe_steps=4, cache_path=str(path))
    lines = path.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split()[0] == key.replace("/S5/", "/S6/")
    assert lines[1].split()[1:4] == [str(x) for x in sched]
