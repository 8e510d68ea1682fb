"""A state's way into the storage of a grid or a batch in one pass, against the
same by torch's copies: every value bit for bit (both only move values), the
padding zero, for both layouts, dense and strided sources, odd widths and
pitches, sources aligned to 8 bytes only, and sources inside the destination."""
import pytest
import torch

from paper_1701_05431_amd import _lib
from paper_1701_05431_amd.solver import Batch, Solver, aligned_pitch, logical, params_from

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def field(nv, ny, cols, kind):
    """An (nv, ny, cols) tensor of distinct values, NaN and infinity among them."""
    g = torch.Generator(device=DEV).manual_seed(nv * 1000003 + ny * 1009 + cols)
    n = (nv + 1) * (ny + 1) * (cols + 4)
    t = torch.randn(n, dtype=torch.float64, device=DEV, generator=g)
    t[n // 3], t[n // 2] = float("nan"), float("inf")
    if kind == "dense":
        return t[:nv * ny * cols].view(nv, ny, cols)
    if kind == "odd":  # 8 bytes off a 16 byte boundary
        return t[1:nv * ny * cols + 1].view(nv, ny, cols)
    if kind == "window":
        return t.view(nv + 1, ny + 1, cols + 4)[1:, 1:, 2:2 + cols]
    if kind == "rows":  # variables inside the rows
        return t[:nv * ny * cols].view(ny, nv, cols).permute(1, 0, 2)
    if kind == "expanded":
        return t[:cols].view(1, 1, cols).expand(nv, ny, cols)
    if kind == "columns":  # not a unit step along x: the general way
        return t[:nv * ny * cols].view(nv, cols, ny).transpose(1, 2)
    raise ValueError(kind)


def by_copies(p, nv, W):
    out = torch.zeros((p.ny, nv, p.ld) if p.layout else (nv, p.ny, p.ld), dtype=torch.float64,
                      device=DEV)
    logical(p, out)[:, :, :W.shape[2]] = W
    return out


def equal(a, b):
    return torch.equal(a.contiguous().view(torch.int64), b.contiguous().view(torch.int64))


@pytest.mark.parametrize("kind", ["dense", "odd", "window", "rows", "expanded", "columns"])
@pytest.mark.parametrize("layout", [0, 1])
def test_a_state_reaches_the_storage(layout, kind):
    for model, nx, ny, ld in [(0, 1, 1, 1), (0, 64, 3, 64), (1, 63, 5, 63), (1, 128, 7, 130),
                              (1, 129, 6, 144), (1, 130, 300, 130), (2, 255, 9, 256),
                              (2, 64, 40, 67)]:
        ug = torch.zeros((2, ny, nx), dtype=torch.float64, device=DEV) if model == 2 else None
        s = Solver(params_from(model=model, nx=nx, ny=ny, ld=ld, layout=layout, bc=1), ug=ug)
        for cols in {nx, ld}:
            print(model, nx, ny, ld, layout, kind, cols, flush=True)
            W = field(s.nv, ny, cols, kind)
            want = by_copies(s.p, s.nv, W)
            s.wa.fill_(7.0)
            s.set_state(W)
            assert s._load(W) == (kind != "columns" or ny == 1 or cols == 1)
            assert equal(s.current_storage(), want)
            out = torch.empty_like(want)
            if s._load(W, out):
                assert equal(out, want)
            assert s.status() == 0  # setting a state checks nothing


@pytest.mark.parametrize("layout", [0, 1])
def test_sources_inside_the_state(layout):
    s = Solver(params_from(model=1, nx=40, ny=40, ld=40, layout=layout, bc=1))
    W = field(4, 40, 40, "dense")
    for view in (lambda w: w, lambda w: w.view(4, 40, 40), lambda w: w.view(40, 4, 40).transpose(0, 1),
                 lambda w: w.view(4, 40, 40)[:1].expand(4, 40, 40)):
        s.set_state(W)
        src = view(s.current_storage())
        if src.shape != (4, 40, 40):
            continue
        want = by_copies(s.p, 4, src.clone())
        s.set_state(src)
        assert equal(s.current_storage(), want)


def test_a_captured_load_reads_its_source_again():
    s = Solver(params_from(model=1, nx=70, ny=50, ld=72, layout=1, bc=1))
    W = field(4, 50, 70, "dense")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        s.set_state(W)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            s.set_state(W)
    for k in range(3):
        W.add_(float(k + 1))
        s.current_storage().zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert equal(s.current_storage(), by_copies(s.p, 4, W))


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("count", [1, 3, 300])
def test_a_batch_of_states(layout, count):
    sizes = [8 + (k * 37) % 91 for k in range(count)]
    plist = [params_from(model=1, bc=1, nx=n, ny=n + 3, layout=layout, cfl=0.45,
                         ld=aligned_pitch(n) if k % 2 else n) for k, n in enumerate(sizes)]
    one, two = Batch(plist), Batch(plist)
    states = []
    for k, n in enumerate(sizes):
        W = field(4, n + 3, n, "odd" if k % 3 else "dense").nan_to_num(0.5, 0.5, 0.5).clone()
        W[0] = 1.0 + W[0].abs()
        W[3] = 30.0 + (W[1:3] ** 2).sum(0)
        states.append(W)
    assert one._load(states)
    two.set_states(iter(states))  # one copy a grid
    assert equal(one.current(), two.current())
    da, db = one.run(6, record_dt=True), two.run(6, record_dt=True)
    assert torch.equal(da, db) and bool((da > 0).all())
    assert equal(one.current(), two.current())
    # views of the batch's own buffer, other types and other streams go the general way
    mine = [one.view(one.current(), k)[:, :, :n] for k, n in enumerate(sizes)]
    assert not one._load(mine)
    assert not one._load([W.float() for W in states])
    with torch.cuda.stream(torch.cuda.Stream()):
        assert not one._load(states)
    if count > 1:
        assert not one._load(states[:-1])
    one.set_states([W.float() for W in states])
    two.set_states(iter([W.float() for W in states]))
    assert equal(one.current(), two.current())
    bad = [W.clone() for W in states]
    bad[-1][0, 2, 3] = float("nan")
    one.set_states(bad)
    torch.cuda.synchronize()
    assert one.sync() == _lib.FVM_ENONFINITE
