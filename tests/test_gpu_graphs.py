"""Captured step and trajectory graphs against the same steps launched one by one: bitwise, and
with the context's own counts, so that a run that never captures or never replays does not pass.

A sequence is captured when it comes back (nse_step: at once from forty fixed-coefficient
steps on), in chunks of ten steps for nse_step; a context keeps eight graphs and remembers the
last eight sequences that ran without one.
"""
import math
import os

import pytest
import torch

import nse_inputs as I
import paper_1009_3308_amd as pkg

pytestmark = pytest.mark.gpu
OMEGA = 2.0 * math.pi
# three groups: blocks of members and a lone member, chains on forked streams
ENSEMBLE = [(63, 0, 1e-4)] * 4 + [(31, 0, 1e-3)] * 3 + [(45, 0, 1e-3)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pkg.LIB_PATH):
        from paper_1009_3308_amd import build
        build.build()
    torch.cuda.set_device(0)


def _history(s, specs, seed=0):
    h = s.new_history()
    for j in range(s.order + 1):
        for i, (N, _, _) in enumerate(specs):
            h[j, s.member_slice(i)] = pkg.to_device(I.member_state(seed + i + 11 * j, N))
    return h


def _forcing(s, specs):
    f = s.new_state()
    for i, (N, _, _) in enumerate(specs):
        f[s.member_slice(i)] = pkg.to_device(I.forcing(N))
    return f


@pytest.mark.parametrize("specs", [ENSEMBLE, [(31, 0, 1e-3)]])
@pytest.mark.parametrize("calls,captured,launched", [
    ((13, 20, 25, 10), 1, 5),   # 10 fixed steps launched, then 2 + 2 + 1 chunks replayed
    ((43, 7, 12), 1, 5),        # 40 fixed steps: captured at once
    ((13, 3, 3), 0, 0),
])
def test_step_graphs_equal_eager_bitwise(specs, calls, captured, launched):
    print(f"case: step graphs {len(specs)} members calls={calls}", flush=True)
    stream = torch.cuda.Stream()
    outs = []
    with torch.cuda.stream(stream):
        for graph in (False, True):
            s = pkg.Sphere(specs, omega=OMEGA, dt=1e-3, graph=graph, stream=stream)
            h, f = _history(s, specs), _forcing(s, specs)
            k, got = 0, []
            for n in calls:
                s.step(h, f, k, n)
                k += n
                got.append(h.clone())
            s.sync()
            assert s.graph_counts() == ((captured, launched) if graph else (0, 0))
            outs.append(got)
            s.close()
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,captured,launched", [(13, 0, 0), (43, 10, 40)])
def test_more_histories_than_the_context_keeps(n, captured, launched):
    # ten histories in turn, twice: short calls never come back in time, long ones are captured
    # at once and evicted before they come back (the second round captures again)
    specs, nhist = [(31, 0, 1e-3)] * 2 + [(20, 0, 1e-3)], 10
    print(f"case: histories n={n}", flush=True)
    stream = torch.cuda.Stream()
    outs = []
    with torch.cuda.stream(stream):
        for graph in (False, True):
            s = pkg.Sphere(specs, omega=OMEGA, dt=1e-3, graph=graph, stream=stream)
            hs, f = [_history(s, specs, i) for i in range(nhist)], _forcing(s, specs)
            for h in hs:
                s.step(h, f, 0, n)
            if graph:
                assert s.graph_counts() == (captured, launched)
            for h in hs:
                s.step(h, f, n, n - 3)
            if graph:
                assert s.graph_counts() == (2 * captured, 2 * launched)
            s.sync()
            outs.append([h.clone() for h in hs])
            s.close()
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("specs", [ENSEMBLE, [(31, 0, 1e-3)]])
def test_trajectory_graphs_equal_eager_bitwise(specs):
    # the same buffers four times: launched, captured and replayed, replayed twice; forward
    # and adjoint, other inputs every time
    n, step0 = 9, 5
    print(f"case: trajectory graphs {len(specs)} members", flush=True)
    s = pkg.Sphere(specs, omega=OMEGA, dt=1e-3, graph=True)
    e = pkg.Sphere(specs, omega=OMEGA, dt=1e-3)
    f = _forcing(s, specs)
    tr, hb = s.new_trajectory(n), s.new_history()
    te, he = e.new_trajectory(n), e.new_history()
    for rep in range(4):
        start, bar = _history(s, specs, 3 * rep), _history(s, specs, 50 + rep)
        for a, t, b in ((s, tr, hb), (e, te, he)):
            t[n:] = start
            b.copy_(bar)
            a.step_trajectory(t, f, step0, n)
            a.step_adjoint_trajectory(t, f, step0, n, b)
        torch.cuda.synchronize()
        assert torch.equal(tr, te) and torch.equal(hb, he), rep
        # (forward and adjoint each)
        assert s.graph_counts() == ((0, 0) if rep == 0 else (2, 2 * rep))
    assert e.graph_counts() == (0, 0)
    s.close()
    e.close()


def test_steps_and_trajectories_inside_the_callers_capture():
    # after a call outside, the sequence has come before: inside a capture of the caller's it
    # has to be recorded, not captured again; the recorded steps replay bitwise, with eager
    # work and synchronisation between the replays
    specs, n = [(31, 0, 1e-3)] * 2 + [(20, 0, 1e-3)], 20
    print("case: caller's capture", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = pkg.Sphere(specs, omega=OMEGA, dt=1e-3, graph=True, stream=stream)
        f = _forcing(s, specs)
        h, h0 = s.new_history(), _history(s, specs)
        tr, hb, bar = s.new_trajectory(n), s.new_history(), _history(s, specs, 40)

        def work():
            s.step(h, f, 3, n)
            s.step_trajectory(tr, f, 3, n)
            s.step_adjoint_trajectory(tr, f, 3, n, hb)

        def reset(seed):
            h.copy_(h0 * (1.0 + 0.1 * seed))
            tr[n:] = h
            hb.copy_(bar * (2.0 - seed))

        reset(0)
        work()
        s.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            work()
        assert s.graph_counts() == (0, 0)
        for seed in range(3):
            reset(seed)
            g.replay()
            stream.synchronize()
            got = (h.clone(), tr.clone(), hb.clone())
            reset(seed)
            for i in range(n):  # one step at a time: no graph
                s.step(h, f, 3 + i, 1)
            e = pkg.Sphere(specs, omega=OMEGA, dt=1e-3, stream=stream)
            e.step_trajectory(tr, f, 3, n)
            e.step_adjoint_trajectory(tr, f, 3, n, hb)
            e.sync()
            e.close()
            for a, b in zip(got, (h, tr, hb)):
                assert torch.equal(a, b), seed
        s.close()
