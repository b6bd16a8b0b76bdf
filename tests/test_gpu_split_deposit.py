"""The staged path's two deposits: one thread per particle (small species) and
tile by tile through LDS (more than 8192 particles plus one per 128 cells).  The current is an exact
integer sum, so a set deposited tile by tile as one species equals, bit for
bit, the same set deposited directly as several small ones; grids with
ragged tiles and axes shorter than a tile, particles in random memory order."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402


def _deposit(grid, pl, parts, bc_x=0):
    """J and the momenta (tag order) after one gather_push + deposit of `parts` species."""
    sim = pic.Simulation(grid.n, grid.d, grid.dt, solver=grid.solver, bc_x=bc_x, max_particles=pl.count)
    F = torch.as_tensor(inputs.random_fields(grid, seed=5, amp=0.5))
    sim.E.copy_(F[:3])
    sim.B.copy_(F[3:])
    for idx in np.array_split(np.arange(pl.count), parts):
        sim.add_species(pl.cell[idx], pl.off[:, idx], pl.u[:, idx], pl.w[idx], pl.id[idx])
    for s in range(parts):
        sim.gather_push(s)
    for s in range(parts):
        sim.deposit(s)
    sim.sync()
    J = sim.J.cpu().numpy()
    sim.close()
    return J


@pytest.mark.parametrize("n,count,bc_x", [((9, 5, 4), 8194, 0), ((8, 8, 8), 20000, 0), ((21, 17, 10), 30000, 0),
                                          ((40, 16, 24), 60000, 0), ((30, 13, 9), 40000, 1)])
def test_tilewise_deposit_equals_direct(n, count, bc_x):
    grid = inputs.Grid(n, (0.25, 0.5, 0.4), 0.24, solver="pd")
    pl = inputs.uniform_random_plasma(grid, ppc=-(-count // grid.ncells), seed=3, temperature_ev=50000.0, ux_amp=0.2)
    pick = np.random.default_rng(4).permutation(pl.count)[:count]
    pl = inputs.Particles(cell=pl.cell[pick].copy(), off=pl.off[:, pick].copy(), u=pl.u[:, pick].copy(),
                          w=pl.w[pick].copy(), id=pl.id[pick].copy())
    pl.cell[::97] = -1                                  # removed particles stay out of the list
    one = _deposit(grid, pl, 1, bc_x)
    many = _deposit(grid, pl, -(-count // 8192), bc_x)  # every species at most 8192: the direct path
    assert np.abs(one).max() > 0
    assert np.array_equal(one, many)
