"""Convolutions whose input channels are shared out over workgroups (small volumes, many channels): remainders of tiles, several channel
blocks, splits and samples, with bias and statistics, forward and data gradient, against 64-bit torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def conv(x, w27):
    D, H, W = x.shape[1:4]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    return sum(xp[:, t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[4]) @ w27[:, t].t()
               for t in range(27)).reshape(*x.shape[:4], -1)


@pytest.mark.parametrize("shape,co", [((1, 4, 8, 16, 128), 64), ((2, 5, 7, 9, 256), 192), ((1, 8, 8, 8, 512), 512), ((3, 3, 5, 6, 256), 64),
                                      ((1, 9, 9, 17, 144), 128), ((2, 8, 8, 8, 128), 256), ((1, 1, 1, 1, 1024), 64), ((1, 16, 16, 16, 192), 256)],
                         ids=str)
def test_split_conv(L, shape, co):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + co)
    ci = shape[4]
    x = torch.randn(shape, generator=g, device="cuda").to(BF)
    dz = torch.randn((*shape[:4], co), generator=g, device="cuda").to(BF)
    w = (torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * (2.0 / (27 * ci)) ** 0.5).to(BF)
    b = torch.randn((co,), generator=g, device="cuda")
    w27 = w.double().reshape(co, 27, ci)
    z, dx, st = torch.empty_like(dz), torch.empty_like(x), torch.empty((shape[0], co, 2), device="cuda")
    L.lamp_conv3d_fwd(x, w, z, bias=b, stats_out=st)
    L.lamp_conv3d_dgrad(dz, w, dx)
    zr, dxr = conv(x, w27) + b.double(), conv(dz, w27.flip(1).permute(2, 1, 0))
    # one rounding to bf16 of fp32 sums
    assert ((z.double() - zr).norm() / zr.norm()).item() <= 2.0 ** -8 and ((dx.double() - dxr).norm() / dxr.norm()).item() <= 2.0 ** -8
    m = z.double().mean((1, 2, 3))
    v = z.double().var((1, 2, 3), unbiased=False)
    r = torch.rsqrt(v + 1e-5)
    # fp32 sums of at most 32 rows, fp64 behind them; the variance is their difference
    assert (st[..., 0] - m).abs().max().item() <= 1e-5
    assert ((st[..., 1] - r) / r).abs().max().item() <= 2.0 ** -20 * ((v + m * m) / (v + 1e-5)).max().item()
