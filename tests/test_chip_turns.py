"""What the host asks of the runtime for runs that keep the state on the chip,
without a GPU: the library runs in a child process on stand-ins of the HIP calls
(tests/emu/hip_calls.cpp) that log every launch, event record and wait. Such
runs wait for all of their workgroups to be resident, so runs that are not
ordered must fit the chip together, whatever the handles of their streams say (a
handle may name another stream than the one it named before); and no stream waits
for another one's work."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

# argv: the stand-ins, a list of actions; prints the log as lists, one per action
CHILD = """
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1])
stub.calls_log.restype = C.c_char_p
from paper_1701_05431_amd import _lib
L = _lib.lib()
grids, logs = {}, []
def grid(name, nx, ny, stream=0, model=1):
    p = _lib.Params(model=model, bc=1, nx=nx, ny=ny, npart_x=1, npart_y=1, ld=nx, layout=0,
                    lx=1.0, ly=1.0, gamma=1.4, ax=1.0, ay=0.5, cfl=0.4)
    h = C.c_void_p()
    code = L.fvm_create(C.byref(p), C.byref(h))
    at = 4096 * (1 + 10 * len(grids))  # never looked at: nothing runs
    grids[name] = h
    return code or L.fvm_bind(h, at, at + 4096, None, at + 8192, stream)
def run(name, steps=20):
    return L.fvm_run_dts(grids[name], steps, 8)
def buffers(n):
    return (C.c_void_p * n)(*range(1 << 20, (1 << 20) + 8 * n, 8))
def ckpt(name, steps, every):
    n = -(-steps // every)
    return L.fvm_run_ckpt(grids[name], steps, every, buffers(n), 8)
def back(name, steps, every):
    n = -(-steps // every)
    return L.fvm_adjoint_run(grids[name], buffers(n), every, 8, steps, 1 << 21, 1 << 22, 1 << 23)
def stream(name, s):
    return L.fvm_set_stream(grids[name], s)
def device(d):
    return stub.calls_device(d) and 0
def finish():
    return stub.calls_finish() and 0
for f, *args in json.loads(sys.argv[2]):
    stub.calls_clear()
    code = globals()[f](*args) if f in ("grid", "run", "ckpt", "back", "stream", "device", "finish") else \\
        getattr(L, f)(grids[args[0]], *args[1:])
    log = [q.split() for q in stub.calls_log().decode().splitlines()]
    logs.append([code, [[q[0]] + [int(x) for x in q[1:]] for q in log]])
print(json.dumps(logs))
"""


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    from paper_1701_05431_amd import _lib
    if not os.path.exists(CLANG):
        pytest.skip("needs the ROCm clang++ for a host build")
    if not os.path.exists(_lib.LIB_PATH):
        from paper_1701_05431_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("calls") / "hip_calls.so")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "emu", "hip_calls.cpp"), "-o", so], check=True)

    def do(*actions):
        first = os.environ.get("LD_PRELOAD")
        env = dict(os.environ, LD_PRELOAD=so + (":" + first if first else ""))
        out = subprocess.run([sys.executable, "-c", CHILD, so, json.dumps(actions)], cwd=ROOT,
                             env=env, check=True, capture_output=True, text=True, timeout=120)
        return json.loads(out.stdout.splitlines()[-1])

    return do


def turns(results):
    """The runs on the chip of a log an action: [(tiles, the runs that are over
    before it starts: by the events, or since the GPU was idle)]. A stream waits
    for events of its own handle only."""
    runs, done, over, of = [], {}, set(), {}
    for code, log in results:
        assert code == 0, results
        if log == ["finish"]:
            over = set(range(len(runs)))
            continue
        if not any(q[0] == "record" for q in log):
            assert all(q[0] in ("graph", "launch") for q in log), log
            continue
        after = set(over)
        first = next(i for i, q in enumerate(log) if q[0] == "launch")
        for what, a, b, _ in log[:first]:
            assert what == "wait" and of[a] == b, log
            after |= done[a]
        assert [q[0] for q in log[first:]] == ["launch", "launch", "record"], log
        _, event, stream, _ = log[-1]
        done[event], of[event] = after | {len(runs)}, stream
        runs.append((log[first][1], after))
    return runs


def test_equal_stream_handles_are_not_the_same_stream(calls):
    """Two runs of the whole chip from one handle: hipStreamPerThread (2) of two
    threads, or a stream made where a destroyed one was."""
    setup = [("grid", "a", 1024, 1024, 2), ("grid", "b", 1000, 1000, 2)]
    got = calls(*setup, ("run", "a"), ("run", "b"), ("run", "a"))[2:]
    assert [r[1] for r in turns(got)] == [set(), {0}, {0, 1}]


def test_runs_stay_off_the_chip_on_another_devices_stream(calls):
    """A stream of another device than the grid's, or another current device:
    the steps are launches on the stream, as without runs on the chip."""
    one, other = 0x00002, 0x10002  # streams of devices 0 and 1
    got = calls(("grid", "a", 1024, 1024, one), ("run", "a"), ("stream", "a", other), ("run", "a"),
                ("device", 1), ("run", "a"), ("stream", "a", one), ("run", "a"), ("device", 0),
                ("run", "a"))
    assert all(code == 0 for code, _ in got)
    steps = [[q[0] for q in log] for (code, log), f in
             zip(got, "grid run stream run device run stream run device run".split()) if f == "run"]
    chip, launches = ["launch", "launch", "record"], ["graph"]
    assert steps[0] == chip and steps[4] == ["wait"] + chip
    assert steps[1] == steps[2] == steps[3] == launches


def width(after, tiles):
    """The most CUs that runs unordered with each other can want at once."""
    n = len(tiles)
    best = 0
    for pick in range(1, 1 << n):
        k = [i for i in range(n) if pick >> i & 1]
        if not any(i in after[j] for i in k for j in k):
            best = max(best, sum(tiles[i] for i in k))
    return best


def test_small_grids_on_many_streams_run_side_by_side(calls):
    streams = range(2, 10)
    got = calls(*[("grid", str(s), 64, 64, s) for s in streams],
                *[("run", str(s)) for s in streams], *[("run", str(s)) for s in streams])
    runs = turns(got[len(streams):])
    # a stream waits for its own runs only
    assert [r[1] for r in runs] == [set()] * 8 + [{k} for k in range(8)]


def test_no_stream_waits_for_another(calls):
    """A run that finds too little of the chip free makes its steps in launches,
    and is on the chip again once the other stream's run is over."""
    kinds = lambda log: [q[0] for q in log]
    chip = ["launch", "launch", "record"]
    setup = [("grid", "big", 1024, 1024, 2), ("grid", "other", 300, 300, 3),
             ("grid", "small", 64, 64, 4), ("grid", "tiny", 48, 48, 5)]
    got = calls(*setup, ("run", "big"), ("run", "other"), ("ckpt", "other", 9, 3),
                ("back", "other", 12, 6), ("fvm_run", "tiny", 9, 0), ("finish",), ("run", "small"),
                ("run", "other"), ("run", "big"), ("finish",), ("run", "big"))[4:]
    assert all(code == 0 for code, _ in got)
    logs = [kinds(log) for _, log in got]
    assert logs[0] == chip
    assert logs[1] == ["graph"]
    assert set(logs[2]) == set(logs[3]) == {"launch"}
    assert logs[4] == ["launch"] * 2 and got[4][1][-1][1] == 1  # (maxima,) one workgroup
    # "other" takes six eighths of the chip, "small" one
    assert logs[6] == logs[7] == chip
    assert logs[8] == ["graph"]
    assert logs[10] == chip


@pytest.mark.parametrize("sizes", [[(1024, 1024), (64, 64), (200, 150), (1024, 1024), (64, 64)],
                                   [(200, 150)] * 6, [(300, 300), (64, 64), (700, 400)],
                                   [(130, 96), (64, 64), (512, 512)]])
def test_unordered_runs_fit_the_chip_together(calls, sizes):
    """Streams taking runs in turn, each stream a handle of its own or all of
    them one, the GPU idle now and then: never more tiles at once than the chip has
    CUs."""
    n = len(sizes)
    order = [(3 * k * k + k) % n for k in range(14)]
    for same in (False, True):
        grids = [("grid", str(k), nx, ny, 2 if same else 2 + k) for k, (nx, ny) in enumerate(sizes)]
        acts = []
        for i, k in enumerate(order):
            acts += [("run", str(k))] + [("finish",)] * (i % 5 == 4)
        got = calls(*grids, *acts)[n:]
        runs = turns([[0, ["finish"]] if a == ("finish",) else r for a, r in zip(acts, got)])
        after = [set(r[1]) for r in runs]
        for a in after:
            for k in list(a):
                a |= after[k]
        assert len(runs) == 14 if same else len(runs) >= 3
        assert 0 < width(after, [r[0] for r in runs]) <= 256


@pytest.mark.parametrize("nx,ny,blocks", [(64, 64, 8), (200, 150, 59), (1024, 1024, 256),
                                          (1054, 1140, 235)])
def test_a_run_that_cannot_have_the_chip_gets_more_than_one_cu(calls, nx, ny, blocks):
    (_, log), = calls(("grid", "a", nx, ny), ("run", "a"))[1:]
    assert [q[0] for q in log] == ["launch", "launch", "record"]
    (_, tiles, _, _), (_, behind, threads, _) = log[:2]
    assert tiles <= 256 and threads == 512
    # pieces of whole rounds of the workgroup's threads cover the cells
    cells = -(-nx * ny // (256 * 512)) * 512
    assert behind == blocks == -(-nx * ny // cells)


def test_short_runs_are_step_launches(calls):
    """Runs on the chip record their end; a launch for each step, or a graph,
    where the run is too short to pay for its start."""
    def on_chip(*actions):
        return [sum(q[0] == "record" for q in log) for _, log in calls(("grid", "a", 1024, 1024),
                                                                       *actions)[1:]]
    for f in ("fvm_run", "fvm_run_fixed"):
        arg = {"fvm_run": 0, "fvm_run_fixed": 1e-5}[f]
        assert on_chip(*[(f, "a", n, arg) for n in (1, 2, 3, 4)]) == [0, 0, 1, 1]
    assert on_chip(*[("run", "a", n) for n in (1, 2, 3, 4)]) == [0, 0, 1, 1]
    ends = on_chip(*[("ckpt", "a", n, 1) for n in (1, 3, 4, 64, 65, 67, 68)])
    assert ends == [0, 0, 1, 1, 1, 1, 2]
    assert on_chip(*[("ckpt", "a", n, 2) for n in (3, 4, 131, 132)]) == [0, 1, 1, 2]
    # states of up to 2^17 doubles start as fast there as a graph does
    small = [("grid", "b", 256, 128), ("run", "b", 1), ("run", "b", 2), ("grid", "c", 256, 129),
             ("run", "c", 2), ("run", "c", 3)]
    assert on_chip(*small) == [0, 1, 1, 0, 0, 1]
    # segments of so many steps, the first recomputed from its checkpoint
    assert on_chip(("back", "a", 8, 2), ("back", "a", 8, 4), ("back", "a", 10, 5)) == [0, 0, 2]


def test_short_runs_of_small_grids_stay_in_one_workgroup(calls):
    for side, steps, one in ((48, 1, True), (48, 2, True), (48, 3, False), (40, 4, True),
                             (40, 5, False), (34, 18, True), (34, 19, False)):
        _, _, (_, log) = calls(("grid", "a", side, side), ("fvm_run", "a", 1, 0),
                               ("fvm_run", "a", steps, 0))
        assert ([q[:2] for q in log] == [["launch", 1]]) == one
        assert (log[-1][0] == "record") != one


def test_a_lane_layout_can_be_taken_back(calls):
    def chip(*actions):
        return [log[-1][0] == "record" for (_, log), (f, *_) in
                zip(calls(("grid", "a", 300, 200), *actions)[1:], actions) if f == "run"]
    lanes = lambda n: ("fvm_set_cells_per_lane", "a", n)
    run = ("run", "a")
    assert chip(run, lanes(1), run, lanes(0), run, lanes(2), lanes(0), run) == [1, 0, 1, 1]
    # a strip shape has no default to go back to; 0 keeps it
    assert chip(("fvm_set_tiling", "a", 8, 2), run, ("fvm_set_tiling", "a", 0, 0), lanes(0),
                run) == [0, 0]
    assert chip(("fvm_set_tiling", "a", 0, 0), run) == [1]
