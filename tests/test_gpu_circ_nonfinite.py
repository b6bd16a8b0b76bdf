"""A quasi-cylindrical particle whose z offset is not a number is reported by
the fused step wherever it sits, in a tile without any field too."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402
from tests.test_gpu_circ import DR, NZ, _seeded_fields, _sim_with  # noqa: E402


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("fused", [True, False])
def test_nan_offset_is_reported(field, fused):
    n = 100
    jr = np.arange(n) % 8
    x = ((jr + 0.5) * DR).astype(np.float32)
    off = np.stack([np.full(n, 0.25, np.float32), x, np.zeros(n, np.float32)])
    off[0, 37] = np.nan
    F = _seeded_fields(78, amp=0.2)
    if not field:
        F[:] = 0.0
    sim = _sim_with(F, (20 + np.arange(n) % 9 + NZ * jr).astype(np.int32), off, np.zeros((3, n), np.float32),
                    np.full(n, 0.5, np.float32), np.arange(n, dtype=np.int32))
    if fused:
        sim.step(1)
    else:
        sim.gather_push(0)
    with pytest.raises(pic.PicError) as e:
        sim.sync()
    assert e.value.status == pic.PIC_ENONFINITE
