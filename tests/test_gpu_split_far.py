"""The staged path's deposit of particles whose cells a caller changed by
several cells after the push: tile by tile (a large species) as one thread per
particle (the same set in small species) deposits them, bit for bit."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402


def _deposit(grid, pl, shift, parts):
    sim = pic.Simulation(grid.n, grid.d, grid.dt, solver="pd", max_particles=pl.count)
    F = torch.as_tensor(inputs.random_fields(grid, seed=5, amp=0.5))
    sim.E.copy_(F[:3])
    sim.B.copy_(F[3:])
    n = grid.n
    for idx in np.array_split(np.arange(pl.count), parts):
        sim.add_species(pl.cell[idx], pl.off[:, idx], pl.u[:, idx], pl.w[idx], pl.id[idx])
    for s in range(parts):
        sim.gather_push(s)
        v = sim.particles(s)
        c, d = v["cell"].long(), torch.as_tensor(shift, device=v["cell"].device)[:, v["id"].long()]
        x, y, z = c % n[0], (c // n[0]) % n[1], c // (n[0] * n[1])
        v["cell"].copy_((x + d[0]) % n[0] + n[0] * ((y + d[1]) % n[1] + n[1] * ((z + d[2]) % n[2])))
    for s in range(parts):
        sim.deposit(s)
    sim.sync()
    J = sim.J.cpu().numpy()
    sim.close()
    return J


@pytest.mark.parametrize("most", [1, 2, 5])
def test_deposit_after_far_moves(most):
    grid = inputs.Grid((21, 17, 16), (0.25, 0.5, 0.4), 0.24, solver="pd")
    pl = inputs.uniform_random_plasma(grid, ppc=3, seed=3, temperature_ev=50000.0, ux_amp=0.2)
    shift = np.random.default_rng(9).integers(-most, most + 1, (3, pl.count))
    one, many = _deposit(grid, pl, shift, 1), _deposit(grid, pl, shift, 3)
    assert np.abs(one).max() > 0 and np.array_equal(one, many)
