"""The fused kernel's queue of cell-crossing particles: plasmas in which nearly
every, some and hardly any particles cross a face per step, with tile
populations around the wavefront and workgroup sizes, against the staged path
(one thread per particle, global atomics) bit for bit."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402


@pytest.mark.parametrize("uth", [5.0, 0.3, 0.001])
@pytest.mark.parametrize("tiling", [dict(threads=256), dict(threads=512), dict(threads=1024),
                                    dict(tile=(5, 3, 7), guard=2, threads=512), dict(tile=(8, 8, 4), threads=1024),
                                    dict(guard=0, threads=1024)])
@pytest.mark.parametrize("count", [1, 63, 65, 1025, 7000])
def test_fused_equals_staged(uth, tiling, count):
    n, d = (17, 16, 9), (0.25, 0.3, 0.3)
    rng = np.random.default_rng(count)
    # half of them in one tile, the rest anywhere
    c = np.stack([np.where(np.arange(count) % 2, rng.integers(0, n[a], count), rng.integers(0, min(8, n[a]), count))
                  for a in range(3)])
    cell = (c[0] + n[0] * (c[1] + n[1] * c[2])).astype(np.int32)
    off = inputs.offset_f32(rng.random((3, count)))
    u = (uth * rng.standard_normal((3, count))).astype(np.float32)
    w = np.full(count, 0.125, np.float32)
    ids = np.arange(count, dtype=np.int32)
    F = torch.as_tensor(inputs.random_fields(inputs.Grid(n, d, 0.24), seed=2, amp=0.2))
    out = []
    for fused in (True, False):
        sim = pic.Simulation(n, d, 0.24, solver="pd", max_particles=count, **(tiling if fused else {}))
        sim.E.copy_(F[:3])
        sim.B.copy_(F[3:])
        sim.add_species(cell, off, u, w, ids)
        for _ in range(2):
            if fused:
                sim.step(1)
            else:
                sim.gather_push()
                sim.deposit()
                sim.field_step()
        p = sim.particles_host()
        o = np.argsort(p["id"])
        out.append([p["cell"][o], p["off"][:, o], p["u"][:, o], sim.J.cpu().numpy(), sim.E.cpu().numpy()])
        sim.close()
    assert np.abs(out[0][3]).max() > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
