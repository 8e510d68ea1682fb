"""The adjoint's inner tiles, which leave out what a boundary needs, against
tiles that all reach from one boundary to the other: one step's multipliers bit
for bit (every face and cell is evaluated with the same arguments, so no
tolerance), for every boundary condition, inner strips next to the last column
among them."""
import pytest
import torch

from paper_1701_05431_amd import inputs
from paper_1701_05431_amd.solver import Solver, params_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("bc", [0, 1, 2])
def test_inner_tiles(model, bc):
    for nx, ny, ld in [(187, 12, 187), (186, 13, 190), (188, 9, 188), (125, 30, 125), (311, 41, 311)]:
        W = (inputs.perturbed_riemann_state(nx, ny, 3) if model == 1
             else inputs.advection_state(nx, ny, 2))
        s = Solver(params_from(model=model, bc=bc, nx=nx, ny=ny, ld=ld, layout=ny % 2, ax=0.8,
                               ay=-0.6, cfl=0.4))
        if bc == 2:
            s.set_boundary_states([[1.0, 0.2, -0.1, 2.6]] * 4 if model == 1 else [[0.3]] * 4)
        lam = torch.randn((s.nv, ny, nx), dtype=torch.float64, device="cuda:0",
                          generator=torch.Generator(device="cuda:0").manual_seed(nx))
        s.set_adjoint_tiling(ny, 1, 1)
        want = s.adjoint_step(W, 1e-3, lam)[:, :, :nx].clone()
        for rows, wpb in [(1, 1), (2, 1), (2, 4), (3, 2), (4, 1), (6, 8)]:
            print(model, bc, nx, ny, rows, wpb, flush=True)
            s.set_adjoint_tiling(rows, wpb, 1)
            assert torch.equal(s.adjoint_step(W, 1e-3, lam)[:, :, :nx], want)
