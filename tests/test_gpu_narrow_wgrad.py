"""Weight gradient of 1 to 4 bf16 input channels: edges of the 8 x 64 tiles and of the walks along d, every channel count, blocks of 32
outputs and remainders, channel slices, accumulation, against 64-bit torch."""
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
    # products of bf16 are exact in fp32; chains of 256 voxels, up to 32 of them and 4 waves added: sqrt of the length times 2^-24; the
    # one added and taken off costs half a unit of the result it is added to
    assert ((dw2.double() - r).norm() / r.norm()).item() <= 2.0 ** -24 * (256 + 36) ** 0.5
    assert ((dw.double() - 1.0 - r).norm() / (r.norm() + 1.0 * r.numel() ** 0.5)).item() <= 2.0 ** -24 * (256 + 36) ** 0.5
