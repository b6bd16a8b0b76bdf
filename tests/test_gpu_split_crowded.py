"""The staged path's tile-wise gather and deposit of crowded tiles (a beam):
tiles of many workgroups, cells on both sides of the number of particles from
which a tile stays in cell order, list windows that end inside, at and just
past a tile's entries.  Against the same set as small species, which take one
thread per particle, bit for bit."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_split_deposit import _deposit  # noqa: E402
from tests.test_gpu_split_gather import _push  # noqa: E402


def _particles(grid, cells, rng):
    """One particle per entry of `cells`, in random memory order."""
    n = len(cells)
    return inputs.Particles(cell=rng.permutation(cells).astype(np.int32), off=inputs.offset_f32(rng.random((3, n))),
                            u=(0.3 * rng.standard_normal((3, n))).astype(np.float32),
                            w=np.full(n, 0.125, np.float32), id=np.arange(n, dtype=np.int32))


@pytest.mark.parametrize("counts", [
    [8300], [12288], [12289],                             # one cell: windows of 1024 entries
    [24] * 350, [25] + [24] * 349,                        # 24 levels, and one particle more
    [4608] + [0] * 19 + [4609],                           # a whole tile, and one particle more
    [4096, 4095, 1, 4097, 3], [8191, 1, 20000], [1] * 5000 + [9000] + [2] * 300])
@pytest.mark.parametrize("start", [0, 3000])
def test_crowded_deposit_equals_direct(counts, start):
    grid = inputs.Grid((25, 18, 16), (0.25, 0.5, 0.4), 0.24, solver="pd")
    rng = np.random.default_rng(len(counts) + start)
    cells = (start + np.repeat(np.arange(len(counts)), counts)) % grid.ncells
    pl = _particles(grid, cells, rng)
    one = _deposit(grid, pl, 1)
    many = _deposit(grid, pl, -(-pl.count // 8192))
    assert np.abs(one).max() > 0 and np.array_equal(one, many)


@pytest.mark.parametrize("spread", [0.0, 0.6, 2.5])
def test_crowded_gather_equals_direct(spread, count=290000):
    grid = inputs.Grid((64, 64, 32), (0.25, 0.5, 0.4), 0.24, solver="pd")
    rng = np.random.default_rng(7)
    c = np.clip((np.array([[31.2], [40.0], [15.9]]) + spread * rng.standard_normal((3, count))).astype(int), 0, 31)
    c[:, ::5] = rng.integers(0, 32, (3, len(c[0, ::5])))  # and a thin background
    pl = _particles(grid, c[0] + 64 * (c[1] + 64 * c[2]), rng)
    whole = _push(grid, pl, np.arange(count), False)
    parts = [_push(grid, pl, i, False) for i in np.array_split(np.arange(count), 2)]
    for k, a in enumerate(whole):
        assert np.array_equal(a, np.concatenate([p[k] for p in parts], axis=-1))
