"""The staged path's tile-wise gather with the absorbing layer, which removes
the particles in its cells: as the same set pushed directly in parts, bit for
bit."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402


def _push(grid, pl, idx, layers):
    sim = pic.Simulation(grid.n, grid.d, grid.dt, solver="pd", max_particles=pl.count)
    sim.set_pml(layers)
    F = torch.as_tensor(inputs.random_fields(grid, seed=5, amp=0.5))
    sim.E.copy_(F[:3])
    sim.B.copy_(F[3:])
    sim.add_species(pl.cell[idx], pl.off[:, idx], pl.u[:, idx], pl.w[idx], pl.id[idx])
    sim.gather_push()
    sim.deposit()
    sim.sync()
    p = sim.particles_host()
    o = np.argsort(p["id"])
    sim.close()
    return [p["id"][o], p["cell"][o], p["off"][:, o], p["u"][:, o]], sim.J.cpu().numpy()


@pytest.mark.parametrize("n", [(64, 48, 48), (41, 65, 50)])
def test_tilewise_gather_with_the_layer(n, layers=9, count=290000):
    grid = inputs.Grid(n, (0.25, 0.5, 0.4), 0.24, solver="pd")
    pl = inputs.uniform_random_plasma(grid, ppc=-(-count // grid.ncells), seed=3, temperature_ev=50000.0, ux_amp=0.2)
    pick = np.random.default_rng(4).permutation(pl.count)[:count]
    pl = inputs.Particles(cell=pl.cell[pick].copy(), off=pl.off[:, pick].copy(), u=pl.u[:, pick].copy(),
                          w=pl.w[pick].copy(), id=np.arange(count, dtype=np.int32))
    whole, J = _push(grid, pl, np.arange(count), layers)
    parts = [_push(grid, pl, i, layers) for i in np.array_split(np.arange(count), 2)]
    assert np.abs(J).max() > 0
    assert 0.1 < (whole[1] == -1).mean() < 0.9          # the layer's particles are gone, the others are not
    for k, a in enumerate(whole):
        assert np.array_equal(a, np.concatenate([p[0][k] for p in parts], axis=-1))
