"""Runs under stream capture: what is recorded is the run, replay after replay,
with eager work between the replays, and a capture leaves the runs of other
threads alone and they it."""
import threading

import pytest
import torch

from paper_1701_05431_amd import inputs
from paper_1701_05431_amd.solver import Batch, Solver, aligned_pitch, params_from

pytestmark = pytest.mark.gpu


def grid(model, nx, ny, layout=1, closure=0):
    ug = None
    if model == 2:
        W, ug = inputs.spray_state(nx, ny, 5)
    elif model == 1:
        W = inputs.perturbed_riemann_state(nx, ny, 3)
    else:
        W = inputs.advection_state(nx, ny, 2)
    p = params_from(model=model, bc=1 if model == 1 else 0, nx=nx, ny=ny, ld=nx, layout=layout,
                    ax=0.8, ay=-0.6, K=0.05, cfl=0.4, closure=closure)
    return Solver(p, ug=ug), torch.from_numpy(W).cuda()


def replays(record, result, want, between):
    """Records record() and compares result() with `want` after each replay."""
    q = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(q):
        with torch.cuda.graph(graph, stream=q):
            record()
        for _ in range(3):
            graph.replay()
            q.synchronize()
            assert torch.equal(result(), want)
            between()
            q.synchronize()


RUNS = {"adaptive": lambda s, dt: s.run(24), "short": lambda s, dt: s.run(2),
        "two": lambda s, dt: (s.run(20), s.run(4)),
        "fixed": lambda s, dt: s.run_fixed(6, dt),
        "checkpoints": lambda s, dt: s.run_ckpt(8, 3)}


@pytest.mark.parametrize("kind", RUNS)
@pytest.mark.parametrize("model,nx,ny,closure", [(0, 48, 40, 0), (1, 200, 150, 0), (1, 300, 260, 0),
                                                 (2, 130, 90, 0), (2, 64, 48, 1)])
def test_a_captured_run_is_the_run(model, nx, ny, closure, kind):
    eager, W = grid(model, nx, ny, closure=closure)
    eager.set_state(W)
    dt = 0.3 * eager.cfl_dt()[0]
    RUNS[kind](eager, dt)
    want = eager.state()
    s, _ = grid(model, nx, ny, closure=closure)
    kept = []  # (torch's buffers of a recorded call live as long as the graph)

    def record():
        s.set_state(W)
        kept.append(RUNS[kind](s, dt))

    replays(record, s.state, want, lambda: eager.run(3))
    assert s.sync() == 0


@pytest.mark.parametrize("per_grid", [False, True])
def test_a_captured_batch_run_is_the_run(per_grid):
    sizes = [20 + 13 * k for k in range(9)]
    plist = [params_from(model=1, bc=1, nx=n, ny=n + 3, layout=1, cfl=0.45, ld=aligned_pitch(n))
             for n in sizes]
    states = [torch.from_numpy(inputs.riemann_state(n, n + 3, k)).cuda()
              for k, n in enumerate(sizes)]
    eager = Batch(plist)
    eager.set_states(states)
    eager.run(5, per_grid=per_grid)
    eager.run(1, per_grid=per_grid)
    want = eager.current().clone()
    q = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(q):
        b = Batch(plist)  # its stream is the one it was made on
        q.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=q):
            b.set_states(states)
            b.run(5, per_grid=per_grid)
            b.run(1, per_grid=per_grid)
        for _ in range(3):
            graph.replay()
            q.synchronize()
            assert torch.equal(b.current(), want)
            eager.run(2)
            torch.cuda.synchronize()


def test_runs_beside_another_threads_capture():
    """A capture that forbids unsafe calls in every thread of the process."""
    (big, V), (small, W), (c, U) = (grid(1, *n) for n in ((1024, 1024), (300, 200), (200, 150)))
    rb, rs, rc = (grid(1, *n)[0] for n in ((1024, 1024), (300, 200), (200, 150)))
    sb, ss, sc = (torch.cuda.Stream() for _ in range(3))
    for s, X, n in ((rb, V, 20), (rs, W, 20), (rc, U, 24)):
        s.set_state(X)
        s.run(n)
    torch.cuda.synchronize()
    go, done = threading.Event(), threading.Event()

    def other():
        torch.cuda.set_device(0)
        go.wait(60)
        for s, X, q in ((big, V, sb), (small, W, ss)):
            with torch.cuda.stream(q):
                s.set_state(X)
                s.run(20)
        done.set()

    t = threading.Thread(target=other)
    t.start()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(sc):
        c.set_state(U)
        sc.synchronize()
        with torch.cuda.graph(graph, stream=sc):
            c.set_state(U)
            c.run(20)
            go.set()
            done.wait(60)
            c.run(4)
    t.join()
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c.state(), rc.state())
    assert torch.equal(big.state(), rb.state())
    assert torch.equal(small.state(), rs.state())
