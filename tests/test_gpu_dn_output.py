"""The denoiser's output stage marches along z over columns of 29 x 13 cells,
4 to 16 planes at a time: sizes at those edges against the FP64 oracle, on
periodic grids and behind a moving window whose storage has wrapped."""
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


def _current(n, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((3, n[2], n[1], n[0])) * SCALE[:, None, None, None]).astype(np.float32)


@pytest.mark.parametrize("n", [(4, 4, 4), (28, 12, 5), (29, 13, 7), (30, 14, 8), (59, 27, 9)])
def test_output_columns_periodic(n):
    d = (0.2, 0.25, 0.3)
    J, P = _current(n, 41), _params(42)
    got = _gpu_filter(pic.Simulation(n, d, 0.05, jpost="denoiser"), J, P)
    ref, _ = O.denoise(J.astype(np.float64), SCALE.astype(np.float64), P, d=d)
    assert rel_l2(got, ref) <= 1e-4


@pytest.mark.parametrize("n", [(29, 14, 6), (33, 13, 9)])
def test_output_columns_window(n):
    d = (0.25, 0.5, 0.5)
    sim = pic.Simulation(n, d, 0.25, solver="pd", bc_x=1, jpost="denoiser", max_particles=1)
    sim.add_empty_species(1)
    sim.set_window(0)
    J, P = _current(n, 43), _params(44)
    sim.set_denoiser(P, SCALE)
    sim.step(7)
    _, origin = sim.window_state()
    assert origin == 7
    got = _gpu_filter(sim, J, P)
    ref, _ = O.denoise(J.astype(np.float64), SCALE.astype(np.float64), P, d=d,
                       bc=("window", "periodic", "periodic"), origin=origin)
    assert rel_l2(got, ref) <= 1e-4
