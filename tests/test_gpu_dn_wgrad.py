"""Weight and bias gradients of the denoiser's training at crop sizes around
its 16 x 4 x 8-cell tiles and the number of persistent workgroups, against an
FP64 pass that applies the library's own bf16 roundings (input, activations,
output gradient, backward signals), so that the sums themselves are compared.
What is left is FP32 accumulation (1e-6) and roundings that it flips: about
2e-6 / 2^-8 of the values, each by 2^-8, 1e-4 in the norm of a signal, which
the cancellation in the W1 sum raises by about ten: 5e-3 bounds it."""
import numpy as np
import pytest

from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1204_0838_amd import pic  # noqa: E402

CELL = (0.25, 0.5, 0.4)


def _bf16(t):
    return t.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _low(f, dim):
    """f at the cell below along dim, zero outside."""
    return torch.cat([torch.zeros_like(f.narrow(dim, 0, 1)), f.narrow(dim, 0, f.shape[dim] - 1)], dim)


def _high(f, dim):
    return torch.cat([f.narrow(dim, 1, f.shape[dim] - 1), torch.zeros_like(f.narrow(dim, 0, 1))], dim)


def _binomial(f):
    for dim in (-1, -2, -3):
        f = 0.5 * f + 0.25 * (_low(f, dim) + _high(f, dim))
    return f


def _reference(J, T, P, scale):
    """Loss and gradients with the roundings of the training pass."""
    W1, b1, W2, b2, W3, b3 = P
    conv, F = torch.nn.functional.conv3d, torch.nn.functional
    s = scale.view(3, 1, 1, 1)
    x = _bf16(J / s)
    a1 = _bf16(F.relu(conv(x[None], W1, b1, padding=1)[0]))
    a2 = _bf16(F.relu(conv(a1[None], W2, b2, padding=1)[0]))
    y = conv(a2[None], W3, b3, padding=1)[0]
    sigma, dim = CELL[0] * float(scale.sum()) / 3.0, (-1, -2, -3)

    def D(comp, a):
        return (y[comp] - _low(y[comp], dim[a])) / CELL[a]

    out = _binomial(J + sigma * torch.stack([D(2, 1) - D(1, 2), D(0, 2) - D(2, 0), D(1, 0) - D(0, 1)]))
    e = (out - T) / s
    g = _binomial(2.0 / e.numel() * e / s)

    def U(comp, a):
        return (_high(g[comp], dim[a]) - g[comp]) / CELL[a]

    dy = _bf16(sigma * torch.stack([U(2, 1) - U(1, 2), U(0, 2) - U(2, 0), U(1, 0) - U(0, 1)]))

    def back(d, W):   # transposed convolution
        return conv(d[None], W.flip(2, 3, 4).transpose(0, 1), padding=1)[0]

    def dW(d, a):
        return conv(a[:, None], d[:, None], padding=1).transpose(0, 1)

    dz2 = _bf16(back(dy, W3)) * (a2 > 0)
    dz1 = _bf16(back(dz2, W2)) * (a1 > 0)
    bias = [d.sum((1, 2, 3)) for d in (dz1, dz2, dy)]
    return float((e * e).mean()), [dW(dz1, x), bias[0], dW(dz2, a1), bias[1], dW(dy, a2), bias[2]]


@pytest.mark.parametrize("crop", [(1, 1, 1), (16, 4, 8), (17, 5, 9), (15, 3, 7), (48, 12, 24), (33, 9, 16)])
def test_gradients_match_the_rounded_pass(crop):
    nx, ny, nz = crop
    gen = torch.Generator().manual_seed(7)
    scale = torch.tensor([0.5, 1.0, 2.0], dtype=torch.float64)

    def normal(shape, amp):
        return _bf16(amp * torch.randn(shape, generator=gen, dtype=torch.float64))

    J = (torch.randn((3, nz, ny, nx), generator=gen) * scale.view(3, 1, 1, 1)).float()
    T = J + 0.5 * (torch.randn(J.shape, generator=gen) * scale.view(3, 1, 1, 1)).float()
    P = [normal((32, 3, 3, 3, 3), 81 ** -0.5), normal((32,), 0.1), normal((32, 32, 3, 3, 3), 864 ** -0.5),
         normal((32,), 0.1), normal((3, 32, 3, 3, 3), 864 ** -0.5), normal((3,), 0.05)]
    tr = pic.DenoiserTrainer(crop, cell=CELL)
    tr.set_params([p.numpy() for p in P], scale.numpy())
    loss, G = tr.grad(J.cuda(), T.cuda())
    ref_loss, ref = _reference(J.double(), T.double(), P, scale)
    assert abs(loss - ref_loss) <= 1e-3 * ref_loss
    for name, g, gr in zip(("W1", "b1", "W2", "b2", "W3", "b3"), G, ref):
        assert np.all(np.isfinite(g)), name
        assert rel_l2(g, gr.numpy()) <= 5e-3, (name, rel_l2(g, gr.numpy()))
