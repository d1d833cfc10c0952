"""fp32 convolutions at the edges of their chunks: whole and ragged chunks of input channels, output channels short of a block, one to three
input channels, channel slices, tensors off 16 bytes, one or several tiles a workgroup, against 64-bit torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def shifted(x, t):
    D, H, W = x.shape[1:4]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    return xp[:, t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[4])


def conv(x, w27):   # w27 [co][27][ci]
    return sum(shifted(x, t) @ w27[:, t].t() for t in range(27)).reshape(*x.shape[:4], -1)


def sliced(t, extra, off):
    n, d, h, w, c = t.shape
    buf = torch.full((n * d * h * w * (c + extra) + off,), float("nan"), device="cuda")
    v = buf[off:].view(n, d, h, w, c + extra)[..., :c]
    v.copy_(t)
    return v


@pytest.mark.parametrize("shape,co,extra,off", [((1, 5, 6, 7, 8), 4, 0, 0), ((2, 7, 5, 9, 16), 12, 4, 0), ((1, 9, 10, 11, 24), 20, 0, 0),
                                                ((1, 4, 5, 6, 48), 64, 0, 0), ((1, 20, 28, 36, 8), 8, 0, 0), ((2, 33, 32, 17, 16), 40, 0, 0),
                                                ((1, 6, 7, 8, 20), 28, 0, 0), ((1, 8, 9, 10, 16), 16, 0, 1), ((2, 6, 5, 4, 1), 5, 0, 0),
                                                ((1, 40, 50, 60, 1), 8, 0, 0), ((1, 12, 13, 14, 2), 40, 2, 0), ((2, 20, 21, 22, 3), 16, 0, 1),
                                                ((1, 30, 31, 33, 3), 33, 1, 0)], ids=str)
def test_f32_chunks(L, shape, co, extra, off):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + co + off)
    ci = shape[4]
    x = sliced(torch.randn(shape, generator=g, device="cuda"), extra, off)
    dz = sliced(torch.randn((*shape[:4], co), generator=g, device="cuda"), extra, off)
    w = torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * (2.0 / (27 * ci)) ** 0.5
    w27 = w.double().reshape(co, 27, ci)
    z, dx = sliced(torch.zeros_like(dz), extra, off), sliced(torch.zeros_like(x), extra, off)
    st, dw = torch.empty((shape[0], co, 2), device="cuda"), torch.empty_like(w)
    L.lamp_conv3d_fwd(x, w, z, stats_out=st)
    L.lamp_conv3d_dgrad(dz, w, dx)
    L.lamp_conv3d_wgrad(x, dz, dw)
    zr = conv(x, w27)
    dxr = conv(dz, w27.flip(1).permute(2, 1, 0))
    dwr = torch.stack([dz.double().reshape(-1, co).t() @ shifted(x, t) for t in range(27)], 1).reshape(w.shape)

    def rel(a, b):
        return ((a.double() - b).norm() / b.norm()).item()

    # chains of 27 * channels products (weight gradient: 128 voxels, and as many again of chains): sqrt of the length times 2^-24
    assert rel(z, zr) <= 2.0 ** -24 * (27 * ci) ** 0.5 + 2.0 ** -24 and rel(dx, dxr) <= 2.0 ** -24 * (27 * co) ** 0.5 + 2.0 ** -24
    assert rel(dw, dwr) <= 2.0 ** -24 * 256 ** 0.5
    m = z.double().mean((1, 2, 3))
    r = torch.rsqrt(z.double().var((1, 2, 3), unbiased=False) + 1e-5)
    assert ((st[..., 0] - m).abs() * r).max().item() <= 1e-6 and ((st[..., 1] - r) / r).abs().max().item() <= 1e-5
