"""Weights repacked for the matrix-core convolutions: one, two, three, four and six chunks of input channels, chunks and blocks that channels
do not fill, blocks of 32 and 64 outputs, forward and data gradient against 64-bit torch."""
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


# 8-deep tiles (128 slices' worth of work) take the taps in the other order
@pytest.mark.parametrize("vol", [(1, 3, 5, 7), (1, 48, 64, 64)], ids=str)
@pytest.mark.parametrize("ci,co", [(16, 32), (32, 64), (48, 96), (64, 32), (96, 64), (40, 72), (8, 8), (128, 160), (24, 128)], ids=str)
def test_repack(L, vol, ci, co):
    g = torch.Generator(device="cuda").manual_seed(ci + 7 * co + vol[1])
    x = torch.randn((*vol, ci), generator=g, device="cuda").to(BF)
    dz = torch.randn((*vol, co), generator=g, device="cuda").to(BF)
    w = (torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * (2.0 / (27 * ci)) ** 0.5).to(BF)
    w27 = w.double().reshape(co, 27, ci)
    z, dx = torch.empty_like(dz), torch.empty_like(x)
    L.lamp_conv3d_fwd(x, w, z)
    L.lamp_conv3d_dgrad(dz, w, dx)
    zr, dxr = conv(x, w27), conv(dz, w27.flip(1).permute(2, 1, 0))
    # one rounding to bf16 of fp32 sums
    assert ((z.double() - zr).norm() / zr.norm()).item() <= 2.0 ** -8 and ((dx.double() - dxr).norm() / dxr.norm()).item() <= 2.0 ** -8
