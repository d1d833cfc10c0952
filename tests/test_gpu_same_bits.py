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
                                             (512, 256, (33, 32, 32), 2), (160, 32, (33, 32, 33), 3), (32, 32, (33, 32, 33), 3)], ids=str)
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


# dgamma of one sample, every rounding of its sum written out: chunks of max(32, V / 1024) rows whatever the width, the row lanes of a
# 256-thread block, each a chain of fused multiply-adds, folded in fp64 (up to 64 channels in 256 / (2 C) shares, rounded to fp32), the
# chunks in fp64.  fp32 tensors: at least four rows to a row lane, fp64 within a chunk.
def dgamma_of(dy, z, mean, rstd, vec):
    v, c = z.shape
    f = np.float32
    rl = 256 // min(c // vec, 256)
    rows = max(32, -(-v // 1024), 4 * rl if vec == 4 else 0)
    chunks = -(-v // rows)
    zh = ((z - mean) * rstd).astype(f).astype(np.float64)
    g = np.zeros((chunks * rows, c)); g[:v] = dy
    h = np.zeros((chunks * rows, c)); h[:v] = zh
    if vec == 4:
        return (g * h).reshape(chunks, rows, c).sum(1).astype(f).astype(np.float64).sum(0).astype(f)
    rounds = -(-rows // rl)
    acc = np.zeros((chunks, rl, c), f)
    for k in range(rounds):
        n = min(rl, rows - k * rl)
        p = [a.reshape(chunks, rows, c)[:, k * rl:k * rl + n] for a in (g, h)]
        acc[:, :n] = (p[0] * p[1] + acc[:, :n].astype(np.float64)).astype(f)
    acc = acc.astype(np.float64)
    shares = 256 // (2 * c) if 2 * c <= 128 else 1
    part = sum(acc[:, s::shares].sum(1).astype(f).astype(np.float64) for s in range(shares))
    return part.astype(f).astype(np.float64).sum(0).astype(f)


@pytest.mark.parametrize("dtype", [torch.float32, BF], ids=["f32", "bf16"])
@pytest.mark.parametrize("c", [8, 16, 24, 48, 64, 128, 256])
@pytest.mark.parametrize("dims", [(16, 13, 17), (33, 32, 37)], ids=str)
def test_backward_sums_order(L, dtype, c, dims):
    g = torch.Generator(device="cuda").manual_seed(c)
    z, dy = (torch.randn((1, *dims, c), generator=g, device="cuda").to(dtype) for _ in range(2))
    st = torch.stack([torch.randn((1, c), generator=g, device="cuda") * 0.1, torch.rand((1, c), generator=g, device="cuda") + 0.5], -1).contiguous()
    be = torch.full((c,), 50.0, device="cuda")   # no element below zero: the mask is not what is looked at
    dz, dga, dbe = torch.empty_like(z), torch.empty((c,), device="cuda"), torch.empty((c,), device="cuda")
    L.lamp_inorm_relu_bwd(dy, z, st, dz, beta=be, dgamma=dga, dbeta=dbe)
    a, b = (t.float().cpu().numpy().reshape(-1, c) for t in (dy, z))
    want = dgamma_of(a, b, st[0, :, 0].cpu().numpy(), st[0, :, 1].cpu().numpy(), 8 if dtype == BF else 4)
    assert np.array_equal(dga.cpu().numpy(), want)
