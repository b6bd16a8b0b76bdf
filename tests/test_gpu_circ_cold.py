"""Quasi-cylindrical fused step in tiles without any field: particles without
momentum are left as they are there, moving ones (and those of zero momentum
with a sign) are not.  Fields in none, one corner or all of the tiles, against
the staged path (one thread per particle) bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_circ import DR, NR, NZ, _seeded_fields, _sim_with  # noqa: E402


@pytest.mark.parametrize("field", ["none", "node", "all"])
@pytest.mark.parametrize("count", [1, 65, 3000])
def test_fused_equals_staged(field, count):
    rng = np.random.default_rng(count)
    r = rng.uniform(0.0, NR - 1.0, count) * DR          # some beyond the wall margin: removed
    th = rng.uniform(0.0, 2 * np.pi, count)
    x, y = (r * np.cos(th)).astype(np.float32), (r * np.sin(th)).astype(np.float32)
    jr = np.floor(np.sqrt(x * x + y * y) / np.float32(DR)).astype(np.int64)
    oz = rng.integers(0, 1 << 23, count).astype(np.float32) * np.float32(2.0 ** -23)
    u = (0.3 * rng.standard_normal((3, count))).astype(np.float32)
    u[:, np.arange(count) % 4 != 0] = 0.0               # three quarters at rest
    u[1, np.arange(count) % 8 == 1] = -0.0
    args = ((rng.integers(0, NZ, count) + NZ * jr).astype(np.int32), np.stack([oz, x, y]), u,
            np.full(count, 0.5, np.float32), np.arange(count, dtype=np.int32))
    F = _seeded_fields(78, amp=0.2)
    if field != "all":
        keep = F[0, 1, 0, 3, 40]
        F[:] = 0.0
        if field == "node":
            F[0, 1, 0, 3, 40] = keep
    out = []
    for fused in (True, False):
        sim = _sim_with(F, *args)
        for _ in range(2):
            if fused:
                sim.step(1)
            else:
                sim.gather_push(0)
                sim.deposit(0)
                sim.field_step()
        p = sim.particles_host(0)
        o = np.argsort(p["id"])
        out.append([p["id"][o], p["cell"][o], p["off"][:, o], p["u"][:, o], sim.J.cpu().numpy(), sim.E.cpu().numpy()])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
