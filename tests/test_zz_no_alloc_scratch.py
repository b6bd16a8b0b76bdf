"""The allocation-free continuity check keeps to the library's own array: not a
byte of the caller's workspace changes."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_zz_no_alloc import _state  # noqa: E402


@pytest.mark.parametrize("n", [(24, 12, 16), (64, 32, 24)])
def test_workspace_is_left_alone(n):
    sim = _state(n, 2, 5, steps=3)
    sim.sync()
    before = sim.workspace.clone()
    r, j = sim.continuity_noalloc(0)
    assert j > 0 and r <= 1e-6 * j
    assert torch.equal(sim.workspace, before)
    sim.close()
