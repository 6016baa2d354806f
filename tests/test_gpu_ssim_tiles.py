"""The SSIM kernels at the edges of their tiles: one valid position, 64-wide x blocks, 22 and
16 y rows, z runs of one to 34 planes (one and two turns of the register ring), rows of one
and several 1024-position chunks, widths that are no multiple of four.  Reference: the same
definition in float64, its gradient by automatic differentiation.  Tolerances as for the
values and gradients of small volumes elsewhere: 1e-5 of the value; the gradient's terms
cancel to about a tenth of their size and pass six rounded 11-tap sums, 1e-4."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(11, 11, 11), (12, 32, 64), (13, 33, 65), (17, 42, 63), (27, 26, 74), (11, 12, 1023), (12, 11, 1034),
          (11, 13, 1036), (11, 11, 2060), (400, 17, 1100)]


def reference(x, y, L):
    t = torch.arange(11, dtype=torch.float64, device=x.device) - 5
    w = torch.exp(-0.5 * (t / 1.5) ** 2)
    w = w / w.sum()

    def blur(v):
        for dim in range(3):
            n = v.shape[dim] - 10
            v = sum(w[k] * v.narrow(dim, k, n) for k in range(11))
        return v
    mx, my, xx, yy, xy = blur(x), blur(y), blur(x * x), blur(y * y), blur(x * y)
    C1, C2 = (0.01 * L) ** 2, (0.03 * L) ** 2
    return ((2 * mx * my + C1) * (2 * (xy - mx * my) + C2) /
            ((mx * mx + my * my + C1) * (xx - mx * mx + yy - my * my + C2))).mean()


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_tiles_against_float64(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    print("\n[gpu ssim tiles]", shape, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    y = torch.rand(shape, device="cuda", generator=gen)
    x = (y + 0.2 * torch.randn(shape, device="cuda", generator=gen)).clamp_min(0)
    s, g = P.dc_ssim(x, y, 1.0, grad=True)
    s2, _ = P.dc_ssim(x, y, 1.0)
    assert torch.equal(s, s2)
    xd = x.double().requires_grad_(True)
    ref = reference(xd, y.double(), 1.0)
    ref.backward()
    assert abs(float(s) - float(ref)) <= 1e-5 * abs(float(ref))
    assert float((g.double() - xd.grad).norm()) <= 1e-4 * float(xd.grad.norm())
