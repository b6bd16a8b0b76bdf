"""The staged path's two gathers: one thread per particle (small species) and
tile by tile through LDS (more than 262144 particles
plus one per 8 cells, on a grid of at least 256 tiles).  A particle's push does not depend on
the others, so a large set pushed tile by tile equals, bit for bit, its parts
pushed directly; grids with ragged tiles, axes shorter than a tile, a window
whose end removes particles, removed cells, random memory order."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402


def _push(grid, pl, idx, window):
    sim = pic.Simulation(grid.n, grid.d, grid.dt, solver=grid.solver, bc_x=int(window), max_particles=pl.count + 1)
    if window:
        sim.add_empty_species(1)
        sim.set_window(0)
        sim.step(6)                                     # fields stay zero, the origin moves
    F = torch.as_tensor(inputs.random_fields(grid, seed=5, amp=0.5))
    sim.E.copy_(F[:3])
    sim.B.copy_(F[3:])
    s = int(window)
    sim.add_species(pl.cell[idx].copy(), pl.off[:, idx].copy(), pl.u[:, idx].copy(), pl.w[idx].copy(),
                    pl.id[idx].copy())
    sim.gather_push(s)
    sim.sync()
    p = sim.particles_host(s)
    o = np.argsort(p["id"])
    sim.close()
    return [p["id"][o], p["cell"][o], p["off"][:, o], p["u"][:, o]]


@pytest.mark.parametrize("n,window", [((64, 64, 32), False), ((57, 50, 60), False), ((4, 130, 140), False),
                                      ((131, 5, 126), True)])
def test_tilewise_gather_equals_direct(n, window, count=290000):
    grid = inputs.Grid(n, (0.25, 0.5, 0.4), 0.25 if window else 0.24, solver="pd")
    pl = inputs.uniform_random_plasma(grid, ppc=-(-count // grid.ncells), seed=3, temperature_ev=50000.0, ux_amp=0.2)
    pick = np.random.default_rng(4).permutation(pl.count)[:count]
    pl = inputs.Particles(cell=pl.cell[pick].copy(), off=pl.off[:, pick].copy(), u=pl.u[:, pick].copy(),
                          w=pl.w[pick].copy(), id=np.arange(count, dtype=np.int32))
    pl.cell[::97] = -1                                  # removed particles are in no tile
    whole = _push(grid, pl, np.arange(count), window)
    parts = [_push(grid, pl, i, window) for i in np.array_split(np.arange(count), 2)]
    ref = [np.concatenate([p[k] for p in parts], axis=-1) for k in range(4)]
    assert (whole[3] != pl.u[:, whole[0]]).any()
    for a, b in zip(whole, ref):
        assert np.array_equal(a, b)
