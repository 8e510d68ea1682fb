"""Runs that keep the whole state in the LDS of all CUs (one launch a run)
against the same runs as step launches: states, dts, dt log, maxima and status
bit for bit (both evaluate every face and update with the same arguments, so no
tolerance), for every model and boundary condition, at the edges of tiles: one
column or row more than a tile, narrower last tiles, fewer rows than waves,
several tiles in each direction, the largest grids that fit and the first that
do not; adaptive, fixed and given dts, checkpointed runs and their backward
pass, runs in a row, and two grids on two streams."""
import threading

import numpy as np
import pytest
import torch

from paper_1701_05431_amd import _lib, inputs
from paper_1701_05431_amd.solver import Solver, fvrun, params_from

pytestmark = pytest.mark.gpu

GH = {0: [[0.3], [0.1], [0.2], [0.4]],
      1: [[1.0, 0.2, -0.1, 2.6], [0.8, -0.1, 0.1, 2.2], [0.9, 0.0, 0.2, 2.4], [1.1, 0.1, 0.0, 2.8]],
      2: [[1.0, 0.45, 0.21, 0.1, 0.05, -0.02]] * 4}


def solvers(model, bc, nx, ny, layout=0, pad=0, **kw):
    """The grid twice: kept on the chip, and as step launches."""
    ug = None
    if model == 2:
        W, ug = inputs.spray_state(nx, ny, 5)
    elif model == 1:
        W = inputs.perturbed_riemann_state(nx, ny, 3)
    else:
        W = inputs.advection_state(nx, ny, 2)
    base = dict(model=model, bc=bc, nx=nx, ny=ny, ld=nx + pad, layout=layout, ax=0.8, ay=-0.6,
                K=0.05, cfl=0.4)
    base.update(kw)
    out = []
    for resident in (True, False):
        s = Solver(params_from(**base), ug=ug)
        s.set_resident_runs(resident)
        if bc == 2:
            s.set_boundary_states(GH[model])
        s.set_state(W)
        out.append(s)
    return out, W


def same(a, b):
    torch.cuda.synchronize()
    assert torch.equal(a.state(), b.state())
    assert a.cfl_dt() == b.cfl_dt()
    assert a.sync() == b.sync()


SHAPES = [(97, 193), (62, 80), (63, 81), (125, 64), (200, 150), (1, 300), (311, 3), (500, 7)]


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("bc", [0, 1, 2])
def test_runs_equal_step_launches(model, bc):
    for n, (nx, ny) in enumerate(SHAPES):
        print(f"model {model} bc {bc} {nx}x{ny}", flush=True)
        (a, b), _ = solvers(model, bc, nx, ny, layout=n % 2, pad=n % 3)
        for steps in (1, 2, 7):
            da, db = a.run(steps, record_dt=True), b.run(steps, record_dt=True)
            assert torch.equal(da, db)
            same(a, b)
        # the state before the last one is in the other buffer
        oa, ob = (s.wb if s.current_storage() is s.wa else s.wa for s in (a, b))
        assert torch.equal(oa, ob)
        dt = 0.3 * b.cfl_dt()[0]
        for s in (a, b):
            s.run_fixed(3, dt)
            s.run_dts([dt, 0.5 * dt, 0.25 * dt, dt])
        same(a, b)


@pytest.mark.parametrize("model,nx,ny", [(0, 64, 80), (0, 72, 72), (0, 96, 96), (1, 32, 32),
                                         (1, 33, 32), (1, 48, 48), (2, 1, 1024), (2, 41, 25),
                                         (2, 39, 39)])
@pytest.mark.parametrize("strips", [False, True])
def test_the_limits_of_one_workgroup(model, nx, ny, strips):
    """The last grids of one workgroup and the first of several; with a strip
    shape asked for, all of them stay in one workgroup."""
    print(model, nx, ny, strips, flush=True)
    for bc in (0, 1, 2):
        (a, b), _ = solvers(model, bc, nx, ny, pad=bc)
        if strips:
            a.set_tiling(8, 4)
        for steps in (1, 8):
            da, db = a.run(steps, record_dt=True), b.run(steps, record_dt=True)
            assert torch.equal(da, db)
            same(a, b)


@pytest.mark.parametrize("model,nx,ny", [(0, 2108, 2400), (1, 1024, 1024), (1, 1054, 1140),
                                         (1, 1056, 1156), (2, 868, 900), (2, 900, 910)])
def test_the_largest_grids(model, nx, ny):
    print(model, nx, ny, flush=True)
    (a, b), _ = solvers(model, 1 if model == 1 else 0, nx, ny, layout=1)
    da, db = a.run(5, record_dt=True), b.run(5, record_dt=True)
    assert torch.equal(da, db)
    same(a, b)


def test_failed_checks_and_bad_states():
    (a, b), W = solvers(1, 1, 130, 90)
    for s in (a, b):
        s.run_fixed(3, 1.0)  # far beyond the CFL bound: the state stays
        assert s.sync() == _lib.FVM_ECFL
        assert np.array_equal(s.state().cpu().numpy(), W)
        assert s.status(clear=True) == _lib.FVM_ECFL
        s.run(2)
        assert s.sync() == 0
    bad = W.copy()
    bad[0, 40, 70] = -1.0
    for s in (a, b):
        s.set_state(bad)
        s.run(3)
        assert s.sync() == _lib.FVM_ENONFINITE


@pytest.mark.parametrize("nsteps,every", [(65, 1), (66, 1), (150, 1), (131, 2), (193, 3), (194, 3)])
def test_more_checkpoints_than_one_launch_saves(nsteps, every):
    (a, b), _ = solvers(1, 1, 70, 90, layout=1)
    (ca, da), (cb, db) = (s.run_ckpt(nsteps, every) for s in (a, b))
    assert torch.equal(da, db) and len(ca) == len(cb)
    assert all(torch.equal(x, y) for x, y in zip(ca, cb))
    same(a, b)


@pytest.mark.parametrize("nsteps", [1, 12])
def test_the_default_checkpoints_change_no_gradient(nsteps):
    (a, b), W = solvers(1, 1, 70, 90, layout=1)
    grads = []
    for s, every in ((a, None), (b, 4)):
        X = torch.from_numpy(W).cuda().requires_grad_(True)
        (fvrun(X, s, nsteps, every) ** 2).sum().backward()
        grads.append(X.grad)
    assert torch.equal(*grads)


def test_gradients_under_a_memory_limit():
    """A process that may use so little memory that every state does not fit, but
    few checkpoints do: they are what it gets."""
    (a, b), W = solvers(1, 1, 700, 700)
    X = torch.from_numpy(W).cuda().requires_grad_(True)
    state = a.wa.numel() * 8
    (fvrun(X, b, 50, 7) ** 2).sum().backward()
    want = X.grad.clone()
    X.grad = None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    have = torch.cuda.memory_reserved() + 32 * state  # (8 + 7 states and some)
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction(have / total)
    try:
        (fvrun(X, a, 50) ** 2).sum().backward()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(X.grad, want)


@pytest.mark.parametrize("model,every", [(1, 1), (1, 4), (2, 3), (0, 5)])
def test_checkpointed_runs_and_gradients(model, every):
    (a, b), W = solvers(model, 0 if model == 2 else 1, 150, 110, layout=1)
    got = []
    for s in (a, b):
        s.set_state(W)
        ck, dts = s.run_ckpt(11, every)
        end = s.state()
        lam = s.adjoint(ck, every, dts, torch.ones_like(end))
        got.append((end, dts, lam.clone(), [c.clone() for c in ck]))
        assert s.sync() == 0
        s.run(3)
    (ea, ta, la, ca), (eb, tb, lb, cb) = got
    assert torch.equal(ea, eb) and torch.equal(ta, tb) and torch.equal(la, lb)
    for x, y in zip(ca, cb):
        assert torch.equal(x, y)
    same(a, b)


def test_two_grids_on_two_streams():
    (a, ra), _ = solvers(1, 1, 700, 700)
    (b, rb), _ = solvers(1, 0, 640, 500)
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(4):
        with torch.cuda.stream(sa):
            a.run(5)
        with torch.cuda.stream(sb):
            b.run(7)
    torch.cuda.synchronize()
    ra.run(20)
    rb.run(28)
    same(a, ra)
    same(b, rb)


def test_small_and_large_grids_on_many_streams():
    """Runs side by side, and large ones that wait for all of them."""
    sizes = [(1, 64, 64), (1, 200, 150), (2, 90, 60), (1, 1024, 1024), (0, 130, 96), (1, 64, 65)]
    pairs = [solvers(m, 0, nx, ny)[0] for m, nx, ny in sizes]
    streams = [torch.cuda.Stream() for _ in sizes]
    torch.cuda.synchronize()
    for k in range(6):
        for (a, _), q in zip(pairs, streams):
            with torch.cuda.stream(q):
                a.run(3 + k)
    torch.cuda.synchronize()
    for a, b in pairs:
        b.run(sum(3 + k for k in range(6)))
        same(a, b)


def test_threads_on_streams_of_one_handle():
    """hipStreamPerThread: one handle, a stream a thread."""
    (a, _), W = solvers(1, 1, 300, 200)
    W = torch.from_numpy(W).cuda()
    a.run(20)
    want = a.current_storage().cpu()
    got = []

    def work():
        torch.cuda.set_device(0)
        (s, _), _ = solvers(1, 1, 300, 200)
        torch.cuda.synchronize()
        # (nothing of torch's own runs on these streams: its allocator takes
        # streams of equal handles for one)
        with torch.cuda.stream(torch.cuda.ExternalStream(2)):
            for _ in range(10):
                s.set_state(W)
                s.run(20)
            status = s.sync()
            torch.cuda.synchronize()
        got.append((status, torch.equal(s.current_storage().cpu(), want)))

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [(0, True)] * 4


def test_a_chosen_strip_shape_still_runs_strips():
    (a, b), _ = solvers(1, 1, 200, 150)
    a.set_tiling(8, 2)
    a.run(4)
    b.run(4)
    same(a, b)


def control(s, area=False):
    """The words in front of the exchange area (workgroups started, decision,
    workgroups done, a wait ran out), or the area behind them."""
    words = s.scratch_view.view(torch.int64)[32:]
    return words[32:] if area else words[:32]


@pytest.mark.parametrize("model,nx,ny", [(0, 150, 130), (1, 200, 150), (2, 130, 70)])
def test_a_run_that_broke_off_is_not_built_upon(model, nx, ny):
    """What a run leaves behind when a wait runs out, written from the host:
    counts part of the way, words that hold a state. No run takes them for its
    own, and after the status has been cleared the grid runs as a new one."""
    (a, b), W = solvers(model, 1, nx, ny, layout=1)
    empty = control(a, area=True).clone()
    used = empty != 0  # (not what rounds the scratch up to 256 bytes)
    for steps in (4, 5):
        a.run(4)
        torch.cuda.synchronize()
        control(a, area=True).copy_(torch.tensor(0.25, dtype=torch.float64).view(torch.int64))
        control(a)[:4] = torch.tensor([7, 1, 3, 1], device="cuda")
        for _ in range(2):
            a.set_state(W)
            a.run(4)
            assert a.sync() == _lib.FVM_EDEVICE
        assert a.status(clear=True) == _lib.FVM_EDEVICE
        assert a.sync() == 0
        assert torch.equal(control(a, area=True)[used], empty[used])
        for s in (a, b):
            s.set_state(W)
        da, db = a.run(steps, record_dt=True), b.run(steps, record_dt=True)
        assert torch.equal(da, db)
        same(a, b)


def no_go(s):
    """The workgroups of the next run will not all start: the decision, taken by
    the host. (Every kernel of the run ends as it does after a real one.)"""
    torch.cuda.synchronize()
    control(s)[1] = 2


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("bc", [0, 1, 2])
def test_runs_that_cannot_have_the_chip(model, bc):
    """The same states, other buffers, dts, logs, maxima and status as step
    launches; nothing is left behind for the next run."""
    for n, (nx, ny) in enumerate([(97, 193), (125, 64), (200, 150), (1, 6100), (1711, 4),
                                  (700, 701)]):
        print(f"model {model} bc {bc} {nx}x{ny}", flush=True)
        (a, b), W = solvers(model, bc, nx, ny, layout=n % 2, pad=n % 3)
        b.set_tiling(8, 1)  # (no run in one workgroup)
        for steps in (3, 4, 7):
            no_go(a)
            da, db = a.run(steps, record_dt=True), b.run(steps, record_dt=True)
            assert torch.equal(da, db)
            same(a, b)
            oa, ob = (s.wb if s.current_storage() is s.wa else s.wa for s in (a, b))
            assert torch.equal(oa, ob)
            assert not control(a)[:10].any()  # (all but the last maxima and dt)
        dt = 0.3 * b.cfl_dt()[0]
        for call in (lambda s: s.run_fixed(3, dt), lambda s: s.run_dts([dt, 0.5 * dt, dt]),
                     lambda s: s.run_fixed(4, 1e3 * dt)):
            no_go(a)
            call(a)
            call(b)
            assert a.status(clear=True) == b.status(clear=True)
            assert torch.equal(a.state(), b.state())
        for s in (a, b):
            s.run(5)  # on the chip again
        same(a, b)


@pytest.mark.parametrize("nsteps,every", [(1, 1), (7, 1), (8, 3), (9, 3), (10, 4), (66, 1),
                                          (131, 2)])
def test_checkpointed_runs_that_cannot_have_the_chip(nsteps, every):
    (a, b), W = solvers(1, 1, 150, 110, layout=1)
    got = []
    for s in (a, b):
        s.set_state(W)
        if s is a:
            no_go(a)
        ck, dts = s.run_ckpt(nsteps, every)
        end = s.state()
        if s is a:
            no_go(a)
        lam = s.adjoint(ck, every, dts, torch.ones_like(end))
        got.append([end, dts, lam.clone()] + [c.clone() for c in ck])
        assert s.sync() == 0
    assert all(torch.equal(x, y) for x, y in zip(*got))
    torch.cuda.synchronize()
    control(a)[:2] = 0  # (a backward pass that recomputes nothing leaves the decision)
    for s in (a, b):
        s.run(3)
    same(a, b)


def test_a_bad_state_that_cannot_have_the_chip():
    (a, b), W = solvers(1, 1, 130, 90)
    bad = W.copy()
    bad[0, 40, 70] = -1.0
    for s in (a, b):
        s.set_state(bad)
        no_go(a)
        s.run(3)
        assert s.sync() == _lib.FVM_ENONFINITE
