"""Field update and binomial filter at the edges of their marches (workgroups
of 64 x 8 columns, 64 x 16 rows for the filter, plane chunks chosen by the
grid's size), periodic and with the window's seam inside the grid, against
the FP64 oracle.  One step is a handful of FP32 operations per value: 1e-6."""
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


@pytest.mark.parametrize("n", [(64, 8, 4), (65, 9, 17), (63, 17, 16), (130, 33, 35), (4, 4, 70)])
@pytest.mark.parametrize("solver,jpost", [("pd", "binomial"), ("yee", "none")])
def test_periodic_field_step(n, solver, jpost):
    grid = inputs.Grid(n, (0.25, 0.5, 0.4), 0.25 if solver == "pd" else 0.15, solver=solver)
    F = inputs.random_fields(grid, seed=7)
    Jr = inputs.random_fields(grid, seed=8)[:3]
    sim = pic.Simulation(n, grid.d, grid.dt, solver=solver, jpost=jpost, max_particles=1)
    sim.E.copy_(torch.as_tensor(F[:3]))
    sim.B.copy_(torch.as_tensor(F[3:]))
    sim.J.copy_(torch.as_tensor(Jr))
    sim.field_step()
    g = O.from_grid(grid)
    J = Jr.astype(np.float64)
    if jpost == "binomial":
        J = O.binomial(g, J)
    E, B = O.field_step(g, F[:3].astype(np.float64), F[3:].astype(np.float64), J)
    for got, ref in ((sim.J, J), (sim.E, E), (sim.B, B)):
        assert rel_l2(got.cpu().numpy(), ref) <= 1e-6


@pytest.mark.parametrize("n", [(64, 9, 8), (67, 16, 19)])
def test_moving_window_seam(n):
    grid = inputs.Grid(n, (0.25, 0.5, 0.4), 0.25, solver="pd", window=True)
    F = inputs.random_fields(grid, seed=7)
    Jr = inputs.random_fields(grid, seed=8)[:3]
    sim = pic.Simulation(n, grid.d, grid.dt, solver="pd", bc_x=1, jpost="binomial", max_particles=1)
    sim.set_window(0)
    sim.E.copy_(torch.as_tensor(F[:3]))
    sim.B.copy_(torch.as_tensor(F[3:]))
    g = O.from_grid(grid)
    E, B = F[:3].astype(np.float64), F[3:].astype(np.float64)
    for k in range(4):                       # the origin moves one cell per step
        sim.J.copy_(torch.as_tensor(np.roll(Jr, k, axis=3)))
        sim.field_step()
        E, B = O.field_step(g, E, B, O.binomial(g, Jr.astype(np.float64)))
        E, B = O.window_shift(g, E, B)
    Ew, Bw, _ = sim.fields_window_order()
    assert sim.window_state()[1] == 4
    assert rel_l2(Ew, E) <= 1e-6 and rel_l2(Bw, B) <= 1e-6
