"""Forward pass of one to three input channels: a view of a wider tensor, on any element, gives the bits of a tensor of its own (loads of a
channel each against loads of a voxel), and reads nothing beside it."""
import pytest
import torch

pytestmark = pytest.mark.gpu
BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


@pytest.mark.parametrize("dtype", [F32, BF], ids=["f32", "bf16"])
@pytest.mark.parametrize("ci", [1, 2, 3])
@pytest.mark.parametrize("dims,co", [((5, 6, 7), 8), ((33, 20, 37), 16), ((40, 41, 50), 40)], ids=str)
def test_views(L, dtype, ci, dims, co):
    if dtype == BF and ci == 1:
        pytest.skip("one bf16 channel has kernels of its own")
    g = torch.Generator(device="cuda").manual_seed(ci + co)
    x = torch.randn((2, *dims, ci), generator=g, device="cuda").to(dtype)
    w = (torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * 0.2).to(dtype)
    z, zv = (torch.empty((2, *dims, co), dtype=dtype, device="cuda") for _ in range(2))
    L.lamp_conv3d_fwd(x, w, z)
    for ld, off in ((ci + 1, 0), (ci + 2, 0)) + (((ci, 1), (ci + 1, 3)) if dtype == F32 else ((ci + 1, 8),)):   # (bf16 starts on 16 bytes)
        buf = torch.full((x.numel() // ci * ld + off,), float("nan"), dtype=dtype, device="cuda")
        v = buf[off:].view(2, *dims, ld)[..., :ci]
        v.copy_(x)
        L.lamp_conv3d_fwd(v, w, zv)
        assert torch.equal(z, zv), (ld, off)
