"""Weight gradient of 1 to 4 bf16 input channels: edges of the 8 x 64 tiles and of the walks along d, every channel count, blocks of 32
outputs and remainders, channel slices, accumulation, against 64-bit torch."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def ref(x, dz):
    D, H, W = x.shape[1:4]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    z = dz.double().reshape(-1, dz.shape[4])
    return torch.stack([z.t() @ xp[:, t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[4])
                        for t in range(27)], 1).reshape(dz.shape[4], 3, 3, 3, x.shape[4])


def sliced(t, extra):
    out = torch.full((*t.shape[:4], t.shape[4] + extra), float("nan"), dtype=t.dtype, device="cuda")[..., :t.shape[4]]
    out.copy_(t)
    return out


@pytest.mark.parametrize("shape,co,xextra,zextra", [((1, 1, 1, 1, 1), 8, 0, 0), ((1, 3, 9, 17, 2), 16, 0, 0), ((2, 2, 8, 64, 1), 32, 0, 0),
                                                    ((1, 5, 7, 65, 2), 24, 1, 8), ((2, 4, 17, 130, 3), 32, 0, 0), ((1, 9, 10, 48, 4), 40, 3, 0),
                                                    ((3, 7, 16, 33, 1), 64, 0, 8), ((1, 6, 11, 31, 2), 96, 0, 0), ((2, 3, 5, 20, 4), 256, 0, 0),
                                                    ((1, 2, 6, 100, 1), 48, 2, 0), ((1, 40, 60, 97, 1), 128, 0, 0), ((2, 64, 40, 50, 2), 16, 0, 0)], ids=str)
def test_narrow_wgrad(L, shape, co, xextra, zextra):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + co)
    x = sliced(torch.randn(shape, generator=g, device="cuda").to(BF), xextra)
    dz = sliced(torch.randn((*shape[:4], co), generator=g, device="cuda").to(BF), zextra)
    dw = torch.ones((co, 3, 3, 3, shape[4]), device="cuda")
    r = ref(x, dz)
    L.lamp_conv3d_wgrad(x, dz, dw, beta=1.0)
    L.lamp_conv3d_wgrad(x, dz, dw2 := torch.full_like(dw, float("nan")))
    # products of bf16 are exact in fp32; at the very most 256 of them in a row and 36 sums of such chains: sqrt of the length times
    # 2^-24 (test_narrow_wgrad_walks has the bound of the chains as they are cut); the one added and taken off costs half a unit of the
    # result it is added to
    assert ((dw2.double() - r).norm() / r.norm()).item() <= 2.0 ** -24 * (256 + 36) ** 0.5
    assert ((dw.double() - 1.0 - r).norm() / (r.norm() + 1.0 * r.numel() ** 0.5)).item() <= 2.0 ** -24 * (256 + 36) ** 0.5


def ref_chunks(x, dz, k=8192):
    n, d, h, w, ci = x.shape
    co, v = dz.shape[4], n * d * h * w
    b = -(-v // k)
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    z = torch.zeros((b * k, co), dtype=torch.float64, device="cuda")
    z[:v] = dz.double().reshape(v, co)
    u = torch.zeros((b * k, 27, ci), dtype=torch.float64, device="cuda")
    for t in range(27):
        u[:v, t] = xp[:, t // 9:t // 9 + d, t // 3 % 3:t // 3 % 3 + h, t % 3:t % 3 + w].reshape(v, ci)
    return torch.bmm(z.view(b, k, co).transpose(1, 2).contiguous(), u.view(b, k, 27 * ci)).sum(0).reshape(co, 3, 3, 3, ci)


# Walks of five slices and more, odd and even lengths and a last one that is shorter, so that every slot of the ring of four slices is
# written over several times; remainders of the 8 x 64 tiles; every instantiation.  steps: slices of the longest walk, as the launch cuts
# d for 768 (512) resident workgroups.
@pytest.mark.parametrize("shape,co,steps", [((12, 23, 61, 97, 1), 16, 6), ((12, 23, 61, 97, 1), 32, 6), ((12, 23, 61, 97, 1), 64, 12), ((12, 35, 50, 70, 2), 16, 9),
                                            ((12, 35, 50, 70, 2), 24, 9), ((8, 27, 50, 70, 2), 64, 7), ((16, 26, 43, 90, 3), 16, 13),
                                            ((6, 17, 43, 90, 3), 40, 6), ((10, 31, 33, 67, 4), 8, 7), ((10, 15, 33, 67, 4), 64, 8)], ids=str)
def test_narrow_wgrad_walks(L, shape, co, steps):
    n, d, h, w, ci = shape
    cb = 2 if ci <= 2 and co > 32 else 1
    cols = n * -(-h // 8) * -(-w // 64) * -(-co // (32 * cb))
    assert -(-d // (256 * (3 if ci <= 2 and cb == 1 else 2) // cols)) == steps >= 5
    g = torch.Generator(device="cuda").manual_seed(ci + co)
    x = torch.randn(shape, generator=g, device="cuda").to(BF)
    dz = torch.randn((*shape[:4], co), generator=g, device="cuda").to(BF)
    dw = torch.empty((co, 3, 3, 3, ci), device="cuda")
    L.lamp_conv3d_wgrad(x, dz, dw)
    r = ref_chunks(x, dz)
    # A chain of l additions carries 2^-24 / sqrt(3) * sqrt(l / 2).  Eight products of 16 voxels in a row; the walk's and the waves' sums
    # in fp64 for one input and for up to 16 outputs, otherwise `steps` of them and two more in fp32; each partial and the result rounded
    # once, as much as two additions each.
    l = 8 + 4 + (0 if ci == 1 or co <= 16 else steps + 4)
    e = ((dw.double() - r).norm() / r.norm()).item()
    assert e <= 2.0 ** -24 / math.sqrt(3.0) * math.sqrt(l / 2.0), e
