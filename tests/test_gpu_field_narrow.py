"""Field step of narrow grids (the B half step takes 16 x 32, 32 x 16 or 64 x 8
columns by the cells along x), with and without the absorbing layer, periodic
and with the window's seam inside the grid, and of a grid of several columns
with the layer, against the FP64 oracle.  A step is a handful of FP32
operations per value: 1e-6 for each, 5e-6 after five."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1204_0838_amd import inputs
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402

D = (0.25, 0.5, 0.4)


def _load(sim, F):
    sim.E.copy_(torch.as_tensor(F[:3]))
    sim.B.copy_(torch.as_tensor(F[3:]))


@pytest.mark.parametrize("n", [(4, 33, 9), (15, 32, 20), (16, 31, 17), (17, 17, 16), (32, 16, 33), (33, 9, 18)])
@pytest.mark.parametrize("solver", ["pd", "yee"])
def test_periodic(n, solver):
    grid = inputs.Grid(n, D, 0.25 if solver == "pd" else 0.15, solver=solver)
    F = inputs.random_fields(grid, seed=7)
    Jr = inputs.random_fields(grid, seed=8)[:3]
    sim = pic.Simulation(n, D, grid.dt, solver=solver, max_particles=1)
    _load(sim, F)
    sim.J.copy_(torch.as_tensor(Jr))
    sim.field_step()
    E, B = O.field_step(O.from_grid(grid), F[:3].astype(np.float64), F[3:].astype(np.float64), Jr.astype(np.float64))
    assert rel_l2(sim.E.cpu().numpy(), E) <= 1e-6 and rel_l2(sim.B.cpu().numpy(), B) <= 1e-6


@pytest.mark.parametrize("n", [(12, 34, 9), (29, 17, 18)])
def test_window_seam(n):
    grid = inputs.Grid(n, D, 0.25, solver="pd", window=True)
    F = inputs.random_fields(grid, seed=7)
    sim = pic.Simulation(n, D, grid.dt, solver="pd", bc_x=1, max_particles=1)
    sim.set_window(0)
    _load(sim, F)
    g = O.from_grid(grid)
    E, B = F[:3].astype(np.float64), F[3:].astype(np.float64)
    for _ in range(5):                       # the origin moves one cell per step
        sim.field_step()
        E, B = O.field_step(g, E, B, np.zeros_like(E))
        E, B = O.window_shift(g, E, B)
    Ew, Bw, _ = sim.fields_window_order()
    assert sim.window_state()[1] == 5
    assert rel_l2(Ew, E) <= 5e-6 and rel_l2(Bw, B) <= 5e-6


@pytest.mark.parametrize("n", [(13, 35, 33), (31, 19, 18), (65, 25, 19), (130, 17, 23)])
@pytest.mark.parametrize("solver,jpost", [("pd", "none"), ("pd", "binomial"), ("yee", "none")])
def test_layer(n, solver, jpost, layers=8):
    dt = 0.25 if solver == "pd" else 0.15
    grid = inputs.Grid(n, D, dt, solver=solver)
    F = inputs.random_fields(grid, seed=7)
    Jr = inputs.random_fields(grid, seed=8)[:3]
    sim = pic.Simulation(n, D, dt, solver=solver, jpost=jpost, max_particles=1)
    sim.set_pml(layers)
    _load(sim, F)
    sim.J.copy_(torch.as_tensor(Jr))
    g = O.make_grid(n, D, dt, solver=solver, yzbc=3)
    P = O.make_pml(g, layers=layers)
    E, B, psi = F[:3].astype(np.float64), F[3:].astype(np.float64), O.zeros_psi(g)
    J = Jr.astype(np.float64)
    for _ in range(5):
        sim.field_step()
        if jpost == "binomial":              # (the filter is periodic in y and z, and J stays filtered)
            J = O.binomial(O.from_grid(grid), J)
        E, B, psi = O.pml_field_step(g, P, E, B, psi, J)
    assert np.abs(psi).max() > 0.01
    assert rel_l2(sim.J.cpu().numpy(), J) <= 5e-6
    assert rel_l2(sim.E.cpu().numpy(), E) <= 5e-6 and rel_l2(sim.B.cpu().numpy(), B) <= 5e-6
