"""Results whose every bit the bf16 nets depend on (a last bit that moves is amplified layer by layer): sums in one order, whatever the
size of the volume or the launch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


# The gradient of a coarse voxel takes its eight fine voxels alone: the first slices of a large volume (several row blocks a wave) and
# these slices as a volume of their own (a row block a wave, units fetched further ahead) give the same bits.
@pytest.mark.parametrize("ci,co,dims,part", [(128, 64, (32, 32, 32), 16), (64, 32, (35, 31, 31), 7), (256, 128, (33, 32, 31), 1), (96, 32, (37, 30, 30), 5),
                                             (512, 256, (33, 32, 32), 2)], ids=str)
def test_convtr_dgrad_small_volume(L, ci, co, dims, part):
    g = torch.Generator(device="cuda").manual_seed(ci + part)
    d, h, w = dims
    dy = torch.randn((1, 2 * d, 2 * h, 2 * w, co), generator=g, device="cuda").to(BF)
    wt = (torch.randn((ci, 2, 2, 2, co), generator=g, device="cuda") * (2.0 / (8 * ci)) ** 0.5).to(BF)
    x = torch.zeros((1, d, h, w, ci), dtype=BF, device="cuda")
    dx = torch.full_like(x, 7.0)
    L.lamp_convtr3d_bwd(x, wt, dy, dx=dx)
    small = torch.full((1, part, h, w, ci), 7.0, device="cuda").to(BF)
    L.lamp_convtr3d_bwd(x[:, :part].contiguous(), wt, dy[:, :2 * part].contiguous(), dx=small)
    assert torch.equal(small, dx[:, :part])
