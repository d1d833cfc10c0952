"""Rounding of the long fp32 sums against 64 bits.

A chain of L additions of terms of either sign into one fp32 accumulator carries a relative error of about
u * sqrt(L / 2), u = 2^-24 / sqrt(3) (the roundings of a sum that grows like sqrt(l)); a sum taken in chains of L whose results are
added in chains of M carries u * sqrt((L + M) / 2).  Partials are added in fp64.  So a bound shows how a kernel cuts a sum."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
U = 2.0 ** -24 / math.sqrt(3.0)


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def chain(l, m=0):
    return U * math.sqrt((l + m) / 2.0)


def rel(a, ref):
    return ((a.double() - ref).norm() / ref.norm()).item()


def rand(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda shape, dtype=F32: torch.randn(shape, generator=g, device="cuda").to(dtype)


def wgrad64(x, dz):
    D, H, W = x.shape[1:4]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    dzt = dz.double().reshape(-1, dz.shape[4]).t().contiguous()
    taps = [xp[:, t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[4]) for t in range(27)]
    return torch.stack([dzt @ t for t in taps], 1).reshape(dz.shape[4], 3, 3, 3, x.shape[4])


# walks of up to about 4096 voxels in chains of 128: at most 32 of them
@pytest.mark.parametrize("shape", [(2, 128, 128, 128, 8, 8), (1, 128, 128, 128, 16, 16), (1, 160, 160, 160, 1, 16), (2, 96, 96, 96, 2, 8),
                                   (2, 96, 96, 96, 4, 24), (1, 96, 95, 97, 32, 32), (2, 64, 48, 80, 16, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_conv3d_wgrad_f32(L, shape):
    n, d, h, w, ci, co = shape
    r = rand(41 + ci)
    x, dz = torch.relu(r((n, d, h, w, ci))), r((n, d, h, w, co))
    dw = torch.empty((co, 3, 3, 3, ci), dtype=F32, device="cuda")
    L.lamp_conv3d_wgrad(x, dz, dw)
    e = rel(dw, wgrad64(x, dz))
    assert e <= chain(128, 32), f"{e:.2e} > {chain(128, 32):.2e}"


# bf16 channel counts outside the multiples of 32: a matrix instruction adds 16 voxels to a chain; `steps` of them (with the additions
# of chains) stand for the chain a thread per weight would have, 256 voxels where 32 MB of partials allow it
@pytest.mark.parametrize("shape,steps", [((2, 64, 80, 96, 2, 16), 19), ((2, 128, 128, 128, 2, 16), 36), ((2, 64, 80, 96, 8, 16), 28),
                                         ((2, 128, 128, 128, 8, 8), 59), ((2, 96, 96, 96, 16, 24), 147), ((2, 96, 96, 96, 8, 40), 122)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_conv3d_wgrad_bf16_ragged(L, shape, steps):
    n, d, h, w, ci, co = shape
    r = rand(51 + ci)
    x, dz = torch.relu(r((n, d, h, w, ci), BF)), r((n, d, h, w, co), BF)
    dw = torch.empty((co, 3, 3, 3, ci), dtype=F32, device="cuda")
    L.lamp_conv3d_wgrad(x, dz, dw)
    e = rel(dw, wgrad64(x, dz))
    assert e <= chain(steps), f"{e:.2e} > {chain(steps):.2e}"


# fp32: slabs of up to about 1024 voxels in chains of 64.  bf16 outside the multiples of 32: matrix instructions in a row that stand for
# a thread per weight's chain, 128 voxels where 32 MB of partials allow it
@pytest.mark.parametrize("dtype,shape,bound", [(F32, (2, 64, 64, 64, 64, 32), (64, 16)), (F32, (1, 100, 100, 100, 8, 4), (64, 8)),
                                               (BF, (2, 64, 64, 64, 16, 8), (8,)), (BF, (1, 100, 100, 100, 16, 8), (16,)),
                                               (BF, (2, 96, 96, 96, 32, 16), (57,))], ids=str)
def test_convtr3d_wgrad(L, dtype, shape, bound):
    n, d, h, w, ci, co = shape
    r = rand(61 + ci)
    x, wt, dy = torch.relu(r((n, d, h, w, ci), dtype)), r((ci, 2, 2, 2, co), dtype), r((n, 2 * d, 2 * h, 2 * w, co), dtype)
    dwt = torch.empty(wt.shape, dtype=F32, device="cuda")
    L.lamp_convtr3d_bwd(x, wt, dy, dwt=dwt)
    cols = dy.reshape(n, d, 2, h, 2, w, 2, co).permute(0, 1, 3, 5, 2, 4, 6, 7).reshape(-1, 8 * co).double()
    e = rel(dwt, (x.double().reshape(-1, ci).t().contiguous() @ cols).reshape(wt.shape))
    assert e <= chain(*bound), f"{e:.2e} > {chain(*bound):.2e}"


def test_convtr3d_bias_gradient_bf16(L):
    """128 values to a product chain, those added in fp64: what rounds is each of the 2048 partials, and the result."""
    r = rand(71)
    x, wt, dy = r((2, 96, 96, 96, 64), BF), r((64, 2, 2, 2, 32), BF), r((2, 192, 192, 192, 32), BF)
    dwt, db = torch.empty(wt.shape, dtype=F32, device="cuda"), torch.empty(32, dtype=F32, device="cuda")
    L.lamp_convtr3d_bwd(x, wt, dy, dwt=dwt, dbias=db)
    e = rel(db, sum(dy[i].sum((0, 1, 2), dtype=torch.float64) for i in range(2)))
    assert e <= math.sqrt(2.0) * U, f"{e:.2e} > {math.sqrt(2.0) * U:.2e}"


# 1024 chunks of 864 rows, 864 / row lanes of them to a thread in two chains, half of the elements masked; then the row lanes in a chain
@pytest.mark.parametrize("c,bound", [(256, (54, 4)), (128, (27, 8))], ids=["256", "128"])
def test_inorm_bwd_sums(L, c, bound):
    r = rand(81)
    z, dy = r((1, 96, 96, 96, c)), r((1, 96, 96, 96, c))
    st = torch.tensor([0.0, 1.0], device="cuda").repeat(1, c, 1).contiguous()   # zhat = z, mask = z > 0, both exact
    dg, db, dz = torch.empty(c, device="cuda"), torch.empty(c, device="cuda"), torch.empty_like(z)
    L.lamp_inorm_relu_bwd(dy, z, st, dz, gamma=torch.ones(c, device="cuda"), beta=torch.zeros(c, device="cuda"), dgamma=dg, dbeta=db)
    g = torch.where(z > 0, dy, torch.zeros_like(dy)).double()
    for got, ref in ((dg, (g * z.double()).sum((0, 1, 2, 3))), (db, g.sum((0, 1, 2, 3)))):
        e = (got.double() - ref).square().mean().sqrt().item() / math.sqrt(z.numel() / c / 2.0)
        assert e <= chain(*bound), f"{e:.2e} > {chain(*bound):.2e}"
