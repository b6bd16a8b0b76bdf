"""The denoiser's last layer streams its input through registers: 14 columns,
4 rows per wavefront, 16 per workgroup, 4 to 16 planes per march.  Sizes at
those edges against the FP64 oracle, and the longer marches of larger grids
against the small grid they repeat (the same sums, so the same bits)."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402
from tests.test_gpu_denoise import SCALE, _gpu_filter, _params  # noqa: E402

D = (0.2, 0.25, 0.3)


def _current(n, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((3, n[2], n[1], n[0])) * SCALE[:, None, None, None]).astype(np.float32)


@pytest.mark.parametrize("n", [(13, 15, 4), (14, 16, 5), (15, 17, 7), (29, 4, 6), (8, 33, 9)])
def test_last_layer_tile_edges(n):
    J, P = _current(n, 31), _params(32)
    got = _gpu_filter(pic.Simulation(n, D, 0.05, jpost="denoiser"), J, P)
    ref, _ = O.denoise(J.astype(np.float64), SCALE.astype(np.float64), P, d=D)
    assert rel_l2(got, ref) <= 1e-4


@pytest.mark.parametrize("reps", [(1, 1, 6), (8, 4, 6), (8, 4, 13)])
def test_longer_marches_repeat_the_small_grid(reps):
    n = (28, 17, 9)
    J, P = _current(n, 33), _params(34)
    small = _gpu_filter(pic.Simulation(n, D, 0.05, jpost="denoiser"), J, P)
    big = tuple(a * b for a, b in zip(n, reps))
    tile = (1, reps[2], reps[1], reps[0])
    got = _gpu_filter(pic.Simulation(big, D, 0.05, jpost="denoiser"), np.tile(J, tile), P)
    assert np.array_equal(got, np.tile(small, tile))
