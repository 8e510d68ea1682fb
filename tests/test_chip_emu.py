"""The kernels of a run that keeps the state on the chip, and of the run by tickets
that takes its place, built for the host (tests/emu/chip_emu.cpp) and run under
AddressSanitizer with exactly sized buffers and a bounds check of the LDS array:
no access outside them, states, the other buffer and saved states equal to the
oracle's (relative L-inf 1e-12, dts within 4 ulp), and no word left behind, for
every model, boundary condition and layout, one tile and several, full and ragged
ones, with all workgroups running, with three and with a single one."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from oracle import fv as orc
from paper_1701_05431_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EMU = os.path.join(ROOT, "tests", "emu")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("needs the ROCm clang++ for a host build")
    out = str(tmp_path_factory.mktemp("chipemu") / "chip_emu")
    subprocess.run([CLANG, "-std=c++20", "-O1", "-g", "-fsanitize=address,bounds",
                    "-fno-sanitize-recover=bounds", "-fno-omit-frame-pointer", "-w",
                    "-ffp-contract=off", "-I", os.path.join(EMU, "shim"),
                    os.path.join(EMU, "chip_emu.cpp"), "-o", out, "-pthread"], check=True)
    return out


def problem(model, nx, ny, seed):
    ug = None
    if model == 0:
        W, ghost = inputs.advection_state(nx, ny, seed), [[0.3], [0.7], [0.5], [0.9]]
    elif model == 1:
        W = inputs.riemann_state(nx, ny, seed)
        ghost = [[1.0, 0.1, -0.2, 2.5], [0.5, -0.1, 0.0, 1.5], [0.8, 0.0, 0.3, 2.0],
                 [0.6, 0.2, 0.1, 1.8]]
    else:
        W, ug = inputs.spray_state(nx, ny, seed)
        ghost = [W[:, 0, 0]] * 4
    return np.ascontiguousarray(W, dtype=np.float64), ug, np.array(ghost)


# nx, ny, pad: one tile; a column more; ragged rows; fewer rows than waves; one column; several of each
SHAPES = [(5, 3, 0), (63, 17, 1), (62, 35, 0), (130, 6, 2), (1, 40, 0), (127, 21, 1)]


@pytest.mark.parametrize("room", [0, 1, 3])
@pytest.mark.parametrize("model", [0, 1, 2])
def test_chip_runs_in_bounds_and_equal_to_the_oracle(emu, tmp_path, model, room):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0:"
                                        "detect_stack_use_after_return=0")

    def run(case):
        n, (bc, (nx, ny, pad)) = case
        layout, every, nsteps = n % 2, (0, 1, 2)[n % 3], 4 + n % 2
        W, ug, ghost = problem(model, nx, ny, n)
        fin, fout = str(tmp_path / f"in{n}"), str(tmp_path / f"out{n}")
        parts = [W.ravel()] + ([ug.ravel()] if ug is not None else []) + [ghost.ravel()]
        np.concatenate(parts).tofile(fin)
        cfl = 0.01 if model == 2 else 0.45  # coarse spray grids: keep the moments well inside
        r = subprocess.run([emu, *map(str, (model, bc, nx, ny, pad, layout, nsteps, every, cfl,
                                            room)), fin, fout],
                           capture_output=True, text=True, env=env, timeout=300)
        if r.returncode != 0:
            return case, r.stdout + r.stderr[-2000:]
        P = orc.params(model, nx, ny, bc=bc, ax=1.0, ay=0.5, K=1.0, theta=0.1, s_eps=0.01, cfl=cfl,
                       ghost=ghost if bc == 2 else None)
        out = np.fromfile(fout)
        saved = (nsteps - 1) // every if every else 0
        fields, rest = out[:(2 + saved) * W.size].reshape((-1,) + W.shape), out[(2 + saved) * W.size:]
        dts, status, full = rest[:nsteps], rest[nsteps], rest[nsteps + 1]
        if status != 0 or full != 0:
            return case, f"status {status}, words left {full}"
        _, odts = orc.run(P, W, nsteps, ug=ug)
        if np.max(np.abs(dts - odts) / np.spacing(odts)) > 4:
            return case, "dts"
        wanted = [(0, nsteps)] + [(2 + q, (q + 1) * every) for q in range(saved)]
        if not every:
            wanted.append((1, nsteps - 1))
        for field, k in wanted:
            ref = orc.run(P, W, k, ug=ug)[0]
            for v in range(W.shape[0]):
                err = np.max(np.abs(fields[field][v] - ref[v]))
                if not err <= 1e-12 * max(np.max(np.abs(ref[v])), 1e-300):
                    return case, f"state {k}, variable {v}: off by {err}"
        return case, None

    cases = list(enumerate((bc, shape) for bc in (0, 1, 2) for shape in SHAPES))
    with ThreadPoolExecutor(max_workers=2) as ex:
        bad = [(c, msg) for c, msg in ex.map(run, cases) if msg]
    assert not bad, bad[:3]
