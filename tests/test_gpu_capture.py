"""Steps captured into a graph: a replay computes what an eager call of the same steps computes from the state
the handle is in, whatever was called on the handle since the capture.  Exact."""
import struct

import numpy as np
import pytest

from paper_2603_25068_amd import workloads as W
from test_gpu_parity import _sim

pytestmark = pytest.mark.gpu

T_AT = 36   # offset of the step counter in a state blob


def _capture(s, st, call):
    import torch
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        call()
    return g


def _replay(g, st):
    import torch
    with torch.cuda.stream(st):
        g.replay()
        torch.zeros(1000, device="cuda").sum()
    st.synchronize()


def _same(s, e, ctx):
    a, b = s.state(), e.state()
    for key in ("status", "link", "pos", "seq"):
        assert np.array_equal(a[key], b[key]), (ctx, key)
    a, b = s.link_state(), e.link_state()
    for key in a:
        assert np.array_equal(a[key], b[key]), (ctx, key)


def _at(s, t):
    """The handle's state as a blob whose step counter reads t, the step that a captured call was recorded at."""
    blob = bytearray(s.full_state())
    struct.pack_into("<i", blob, T_AT, t)
    return bytes(blob)


@pytest.mark.parametrize("nx,n", [(4, 3), (4, 4), (9, 3), (9, 4)])
@pytest.mark.parametrize("at", [50, 51])
def test_replays_after_any_eager_call(nx, n, at):
    """Eager calls between replays: rollouts of odd and even length, a reset, a reset with a prefix of either
    parity, a restored state.  One network in a single workgroup, one with a launch per step."""
    import torch
    w = W.random_small(6, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st), _sim(w)
    s.step(at)
    g = _capture(s, st, lambda: s.step(n))
    kept = s.full_state()

    def again(k):
        s.reset()
        s.step(k)

    between = [lambda: None, lambda: s.step(1), lambda: s.step(2), lambda: s.step(7), s.reset, lambda: again(at),
               lambda: again(at + 1), lambda: again(at), lambda: s.set_full_state(kept), lambda: again(1), lambda: again(50)]
    for k, call in enumerate(between):
        call()
        e.set_full_state(_at(s, at))
        e.step(n)
        _replay(g, st)
        _same(s, e, k)


@pytest.mark.parametrize("nx", [4, 9])
def test_eager_steps_after_replays(nx):
    """The state that a replay leaves is the one that later eager calls step, read and save."""
    import torch
    w = W.random_small(7, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st), _sim(w)
    s.step(31)
    g = _capture(s, st, lambda: s.step(5))
    for k in (1, 2, 3):
        s.reset()
        s.step(31)
        _replay(g, st)
        e.reset()
        e.step(36)
        _same(s, e, k)
        s.set_full_state(_at(s, 36))
        s.step(k)
        e.step(k)
        _same(s, e, k)


@pytest.mark.parametrize("record", [False, True])
@pytest.mark.parametrize("nx,n", [(4, 3), (9, 4)])
def test_capture_as_the_first_rollout(nx, n, record):
    """Eager steps between the capture of a new handle's first steps and their first replay."""
    import torch
    w = W.random_small(8, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st, record=record), _sim(w)
    g = _capture(s, st, lambda: s.step(n))
    s.reset()
    for k in range(3):
        s.step(2 + k)
        e.step(2 + k)
        _same(s, e, k)
        e.set_full_state(_at(s, 0))
        e.step(n)
        _replay(g, st)
        _same(s, e, k)
        s.reset()
        e.reset()


@pytest.mark.parametrize("nx", [4, 9])
def test_replays_after_a_schedule_change(nx):
    """Lane groups set between the capture and a replay (a network that leaves and enters the one-workgroup
    form), and two graphs captured under different ones replayed in turn."""
    import torch
    w = W.random_small(9, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st), _sim(w)
    s.step(20)
    s.set_schedule(8, 8, 8)
    g0 = _capture(s, st, lambda: s.step(3))
    s.set_schedule(32, 64, 16)
    g1 = _capture(s, st, lambda: s.step(2))
    s.set_full_state(_at(s, 20))
    for k, (sched, g, at, n) in enumerate([((32, 64, 16), g1, 23, 2), ((64, 64, 8), g0, 20, 3), ((8, 8, 8), g1, 23, 2),
                                           ((16, 16, 16), g0, 20, 3)]):
        s.set_schedule(*sched)
        s.step(1)
        e.set_full_state(_at(s, at))
        e.step(n)
        _replay(g, st)
        _same(s, e, k)


@pytest.mark.parametrize("nx", [4, 9])
def test_captured_gradients_replay(nx):
    """A rollout and its adjoint in one graph, replayed from the start state after eager rollouts, gradients of
    other groups and a schedule change; bitwise the eager gradients."""
    import torch
    w = W.random_small(10, nx=nx, ny=nx, n_agents=20 * nx * nx, rates=True, steps=120)
    groups = ("free_speed", "jam_density", "cap_mult", "beta")
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st, record=True, ckpt_every=25, tape_windows=4), _sim(w, record=True, ckpt_every=25)
    out = {}

    def call():
        s.step(120)
        out.update(s.backward_device(gT=gT, groups=groups))

    gT = torch.full((1,), 0.3, dtype=torch.float64, device="cuda")
    e.rollout()
    want = e.backward(gT=[0.3], groups=groups)
    torch.cuda.synchronize()
    g = _capture(s, st, call)
    between = [lambda: None, lambda: s.step(33), lambda: (s.rollout(), s.backward(gT=[0.3], groups=("free_speed", "alpha"))),
               lambda: (s.set_schedule(16, 64, 16), s.step(1))]
    for k, f in enumerate(between):
        s.reset()
        f()
        s.reset()
        _replay(g, st)
        e.reset()
        e.rollout()
        _same(s, e, k)
        for name in groups:
            assert np.array_equal(out[name].cpu().numpy(), want[name]), (k, name)


@pytest.mark.parametrize("nx", [4, 9])
def test_replays_after_a_placement(nx):
    """Agents placed after the capture: out of position order (the second stands still on the entry slot behind the
    first while others stand in front of them, and the last one has arrived), in order, and none."""
    import torch
    w = W.random_small(11, nx=nx, ny=nx, n_agents=25 * nx * nx, rates=True, steps=120, lanes_max=3)
    st = torch.cuda.Stream()
    s, e = _sim(w, stream=st), _sim(w)
    g = _capture(s, st, lambda: s.step(7))
    links = np.repeat(np.arange(w.net.n_links), 4)
    pos = np.stack([np.full(w.net.n_links, 3.0), np.full(w.net.n_links, 1.0), 0.5 * w.net.length, w.net.length], 1)
    for k, x4 in enumerate([pos, None, pos[:, ::-1][:, [0, 1, 3, 2]], pos]):
        for x in (s, e):
            x.reset()
            if x4 is not None:
                x.place(np.arange(len(links)), links, x4.ravel())
        e.step(7)
        _replay(g, st)
        _same(s, e, k)
