"""The two-stage diagnostics over more items than their workgroups take in one
pass (262144 threads, four particles each in flight) and more partials than
the combining wavefront takes at once, with removed particles among them:
counts exactly, sums to 1e-12 of numpy's FP64."""
import numpy as np
import pytest

from paper_1204_0838_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402

N, D = (80, 64, 60), (0.25, 0.5, 0.4)
COUNT = 1100003


@pytest.fixture(scope="module")
def loaded():
    rng = np.random.default_rng(12)
    cell = rng.integers(0, N[0] * N[1] * N[2], COUNT).astype(np.int32)
    cell[::37] = -1
    off = inputs.offset_f32(rng.random((3, COUNT)))
    u = (0.4 * rng.standard_normal((3, COUNT))).astype(np.float32)
    w = (0.05 + rng.random(COUNT)).astype(np.float32)
    F = inputs.random_fields(inputs.Grid(N, D, 0.2), seed=4, amp=2.0)
    sim = pic.Simulation(N, D, 0.2, solver="pd", max_particles=COUNT)
    sim.add_species(cell, off, u, w, np.arange(COUNT, dtype=np.int32))
    sim.E.copy_(torch.as_tensor(F[:3]))
    sim.B.copy_(torch.as_tensor(F[3:]))
    sim.J.copy_(torch.as_tensor(F[1:4]))
    live = cell >= 0
    c = cell[live].astype(np.int64)
    return {"sim": sim, "F": F.astype(np.float64), "u": u[:, live].astype(np.float64), "w": w[live].astype(np.float64),
            "y": (c // N[0] % N[1] + off[1, live].astype(np.float64)) * D[1],
            "z": (c // (N[0] * N[1]) + off[2, live].astype(np.float64)) * D[2]}


def _close(a, b):
    return abs(a - b) <= 1e-12 * abs(b)


def test_reduce(loaded):
    got, dv = loaded["sim"].reduce(), D[0] * D[1] * D[2]
    u2 = (loaded["u"] ** 2).sum(axis=0)
    assert got["n_particles"] == len(loaded["w"])
    assert _close(got["charge"], -loaded["w"].sum() * dv)
    assert _close(got["e_kin"], (loaded["w"] * (u2 / (np.sqrt(1 + u2) + 1))).sum() * dv)
    assert _close(got["e_field"], 0.5 * (loaded["F"] ** 2).sum() * dv)
    assert got["max_abs_J"] == np.abs(loaded["F"][1:4]).max()


@pytest.mark.parametrize("quantity,lo,hi", [(0, 0.0, 0.6), (1, -1.0, 1.0)])
@pytest.mark.parametrize("nbins", [1, 57, 2048])
def test_spectrum(loaded, quantity, lo, hi, nbins):
    charge, count = loaded["sim"].spectrum(0, quantity, lo, hi, nbins)
    u2 = (loaded["u"] ** 2).sum(axis=0)
    v = u2 / (np.sqrt(1 + u2) + 1) if quantity == 0 else loaded["u"][0]
    b = np.floor((v - lo) / (hi - lo) * nbins)
    b = b[(b >= 0) & (b < nbins)].astype(np.int64), (b >= 0) & (b < nbins)
    ref = np.bincount(b[0], minlength=nbins)
    refq = np.bincount(b[0], weights=loaded["w"][b[1]], minlength=nbins) * D[0] * D[1] * D[2]
    # (a value within an FP64 rounding of a bin's edge may fall to either side)
    assert np.abs(count - ref).sum() <= 2 and count.sum() == ref.sum()
    same = count == ref
    assert np.abs(charge[same] - refq[same]).max() <= 1e-12 * refq.sum()


def test_beam_moments(loaded):
    got = loaded["sim"].beam_moments(0, 0.3)
    k = loaded["u"][0] > np.float64(0.3)
    w, u = loaded["w"][k], loaded["u"][:, k]
    assert got["count"] == int(k.sum())
    assert _close(got["mean_ux"], (w * u[0]).sum() / w.sum())
    for a, r in ((0, loaded["y"][k]), (1, loaded["z"][k])):
        assert _close(got["mean_r"][a], (w * r).sum() / w.sum())
        # (a difference of squares: 1e-12 of the squares)
        var = (w * r * r).sum() / w.sum() - ((w * r).sum() / w.sum()) ** 2
        assert abs(got["rms_r"][a] ** 2 - var) <= 1e-12 * (w * r * r).sum() / w.sum() * 2


def test_field_moments(loaded):
    got = loaded["sim"].field_moments()
    stag = (0.5, 0.0, 0.0, 0.0, 0.5, 0.5)
    x = np.stack([(np.arange(N[0]) + s) * D[0] for s in stag])[:, None, None, :]
    e = 0.5 * loaded["F"] ** 2 * (D[0] * D[1] * D[2])
    for a, ref in enumerate(((e).sum(), (e * x).sum(), (e * x * x).sum())):
        assert _close(got[a], ref)
