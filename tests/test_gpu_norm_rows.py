"""InstanceNorm + ReLU forward and backward where the rows of a block are cut to whole lines (3, 6, 12 pieces a voxel), with and without
gamma / beta, accumulation, several samples, channel slices and tensors off 16 bytes, against 64-bit torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def slice_of(t, extra, off):
    """The values of t as a channel slice of a wider buffer, `off` elements behind its start."""
    n, d, h, w, c = t.shape
    buf = torch.zeros((n * d * h * w * (c + extra) + off,), dtype=t.dtype, device="cuda")
    v = buf[off:].view(n, d, h, w, c + extra)[..., :c]
    v.copy_(t)
    return v


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape,affine,extra,off", [((2, 5, 7, 9, 24), True, 0, 0), ((1, 13, 12, 11, 48), True, 8, 0), ((3, 4, 5, 6, 96), True, 0, 0),
                                                    ((2, 3, 5, 7, 8), True, 0, 0), ((1, 40, 41, 43, 16), False, 0, 0), ((2, 6, 7, 5, 12), True, 0, 1),
                                                    ((1, 2, 2, 2, 40), True, 0, 0), ((2, 9, 8, 7, 72), False, 0, 3),
                                                    ((2, 6, 5, 7, 64), False, 0, 0), ((1, 6, 5, 7, 256), True, 0, 0), ((3, 7, 8, 9, 8), False, 8, 0)], ids=str)
def test_inorm_relu_rows(L, dtype, shape, affine, extra, off):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + extra)
    n, c = shape[0], shape[4]
    z, dy = (slice_of(torch.randn(shape, generator=g, device="cuda").to(dtype), extra, off) for _ in range(2))
    y, dz = (slice_of(torch.zeros(shape, dtype=dtype, device="cuda"), extra, off) for _ in range(2))
    ga = torch.rand((c,), generator=g, device="cuda") + 0.5 if affine else None
    be = torch.rand((c,), generator=g, device="cuda") - 0.5 if affine else None
    st, dga, dbe = torch.empty((n, c, 2), device="cuda"), torch.ones((c,), device="cuda"), torch.full((c,), 2.0, device="cuda")
    L.lamp_inorm_relu(z, y, st, gamma=ga, beta=be)
    L.lamp_inorm_relu_bwd(dy, z, st, dz, gamma=ga, beta=be, dgamma=dga, dbeta=dbe, beta_acc=1.0)
    z64 = z.double().requires_grad_(True)
    p = [(ga if affine else torch.ones((c,), device="cuda")).double().requires_grad_(True),
         (be if affine else torch.zeros((c,), device="cuda")).double().requires_grad_(True)]
    m = z64.mean((1, 2, 3), keepdim=True)
    u = (z64 - m) * torch.rsqrt(((z64 - m) ** 2).mean((1, 2, 3), keepdim=True) + 1e-5) * p[0] + p[1]
    ref = torch.autograd.grad(torch.relu(u), [z64] + p, dy.double())

    def rel(a, b):
        return ((a.double() - b).norm() / b.norm()).item()

    # bf16: one rounding of each stored value, 2^-9; fp32: sums of at most 70 thousand rows in short chains, and coefficients that
    # carry a few roundings, 16 of 2^-24 at most.  (The variance is a difference of fp32 sums and loses mean^2 / variance: eight voxels
    # keep that below 4 or so, two do not, 3.6e-5 was seen.)
    tol = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -20
    assert rel(y, torch.relu(u).detach()) <= tol
    assert rel(dz, ref[0]) <= tol
    # the sums themselves are fp32 on either storage type; accumulated onto 1 and 2
    assert rel(dga, ref[1] + 1.0) <= 2.0 ** -20 and rel(dbe, ref[2] + 2.0) <= 2.0 ** -20
