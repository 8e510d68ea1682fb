"""The speed pass over a state (one grid, and all grids of a batch in one
launch): the largest cell is found wherever it lies, at widths around the
64-cell pieces a wave takes and heights around its share of them. The spray's
speed is q / m_{2/2}, exact at m_{2/2} = 1, so the maxima are compared exactly;
a batch's dts are those of its grids alone, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1701_05431_amd import inputs
from paper_1701_05431_amd.solver import Batch, Solver, params_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 300), (63, 5), (64, 8), (65, 33), (129, 513),
                                   (700, 700), (2100, 40)])
def test_the_largest_speed_is_found(nx, ny):
    r = np.random.default_rng(nx * 1000 + ny)
    for layout, pad in ((0, 0), (1, 3)):
        W = np.ones((6, ny, nx))
        W[4:] = 1e-3 * r.uniform(-1, 1, (2, ny, nx))
        s = Solver(params_from(model=2, bc=0, nx=nx, ny=ny, ld=nx + pad, layout=layout),
                   ug=np.zeros((2, ny, nx)))
        for j, i in {(0, 0), (ny - 1, nx - 1), (ny - 1, 0), (ny // 2, nx // 3)}:
            V = W.copy()
            V[4, j, i], V[5, ny - 1 - j, i] = -2.5, 1.25
            s.set_state(V)
            _, sx, sy = s.cfl_dt()
            assert (sx, sy) == (2.5, 1.25), (layout, j, i)


@pytest.mark.parametrize("rows,waves", [(32, 2), (8, 1), (256, 8)])
def test_batch_dts_are_the_grids_own(rows, waves):
    sizes = [(64, 64), (1, 9), (257, 40), (130, 300), (31, 1), (512, 512)]
    plist = [params_from(model=1, bc=1, nx=nx, ny=ny, ld=nx + 1) for nx, ny in sizes]
    states = [inputs.riemann_state(nx, ny, k) for k, (nx, ny) in enumerate(sizes)]
    b = Batch(plist)
    b.set_tiling(rows, waves)
    b.set_states(states)
    dts = b.run(1, record_dt=True)[0].cpu()
    for k, (p, W) in enumerate(zip(plist, states)):
        s = Solver(p)
        s.set_state(W)
        assert s.cfl_dt()[0] == float(dts[k]), k
    assert b.sync() == 0
