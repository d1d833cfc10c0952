"""Transposed convolution on the bf16 kernels that walk groups and chunks of voxels: remainders of groups, chunks and walks, every weight
depth, channel slices, accumulation and missing outputs, against 64-bit torch."""
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


def ref(x, wt, b, dy):
    n, d, h, w, ci = x.shape
    co = wt.shape[4]
    x, wt, b, dy = (t.double().requires_grad_(True) if i < 3 else t.double() for i, t in enumerate((x, wt, b, dy)))
    y = (x.reshape(-1, ci) @ wt.reshape(ci, 8 * co)).reshape(n, d, h, w, 2, 2, 2, co)
    y = y.permute(0, 1, 4, 2, 5, 3, 6, 7).reshape(n, 2 * d, 2 * h, 2 * w, co) + b
    return [y.detach()] + list(torch.autograd.grad(y, [x, wt, b], dy))


def rel(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


def sliced(t, extra):
    if not extra:
        return t.contiguous()
    out = torch.zeros((*t.shape[:4], t.shape[4] + extra), dtype=t.dtype, device="cuda")[..., :t.shape[4]]
    out.copy_(t)
    return out


# 1, 31, 33 voxels and walks that end inside a group or chunk; 17000 voxels: a few
# workgroups take a second chunk (test_convtr_long_walks has walks of many); weights off 16 bytes and 48
# input channels take the older kernels; 2 x 5 x 6 x 7 x 256 the unit-at-a-time kernel and the data gradient of small volumes
@pytest.mark.parametrize("shape,co,extra,woff", [((1, 1, 1, 1, 64), 32, 0, 0), ((1, 1, 1, 31, 64), 32, 8, 0), ((1, 3, 1, 11, 64), 32, 0, 0), ((2, 5, 7, 13, 64), 32, 0, 0),
                                                 ((1, 20, 25, 34, 64), 32, 0, 0), ((1, 3, 5, 7, 16), 8, 0, 0), ((2, 4, 5, 9, 32), 16, 8, 0),
                                                 ((1, 5, 6, 7, 128), 64, 0, 0), ((1, 3, 4, 5, 32), 24, 0, 0), ((1, 3, 4, 11, 16), 40, 8, 0),
                                                 ((1, 4, 5, 6, 64), 32, 0, 1), ((1, 4, 5, 6, 48), 32, 0, 0), ((2, 5, 6, 7, 256), 128, 0, 0),
                                                 ((2, 3, 3, 3, 64), 64, 0, 0), ((1, 3, 5, 7, 32), 32, 8, 0), ((2, 3, 5, 7, 64), 16, 0, 0),
                                                 ((1, 1, 1, 31, 32), 16, 8, 0), ((2, 11, 12, 13, 32), 16, 0, 0)], ids=str)
def test_convtr_walks(L, shape, co, extra, woff):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + co)
    n, d, h, w, ci = shape

    def rnd(s):
        return torch.randn(s, generator=g, device="cuda")

    x, dy = sliced(torch.relu(rnd(shape)).to(BF), extra), sliced(rnd((n, 2 * d, 2 * h, 2 * w, co)).to(BF), extra)
    buf = torch.zeros((ci * 8 * co + 8,), dtype=BF, device="cuda")
    wt = buf[woff:woff + ci * 8 * co].view(ci, 2, 2, 2, co)
    wt.copy_(rnd(wt.shape) * (2.0 / (8 * ci)) ** 0.5)
    b = rnd((co,)) * 0.1
    y, dx = sliced(torch.full((n, 2 * d, 2 * h, 2 * w, co), 7.0, device="cuda").to(BF), extra), sliced(torch.full(shape, 7.0, device="cuda").to(BF), extra)
    dwt, db = torch.ones((ci, 2, 2, 2, co), device="cuda"), torch.ones((co,), device="cuda")
    L.lamp_convtr3d(x, wt, y, bias=b)
    L.lamp_convtr3d_bwd(x, wt, dy, dx=dx, dwt=dwt, dbias=db, beta=1.0)
    r = ref(x, wt, b, dy)
    # one rounding to bf16; fp32 sums of at most 17000 products in chains of 512 (weights) or fewer: sqrt(chain) * 2^-24 and margin
    assert rel(y, r[0]) <= 2.0 ** -8 and rel(dx, r[1]) <= 2.0 ** -8
    assert rel(dwt - 1.0, r[2]) <= 1e-5 and rel(db - 1.0, r[3]) <= 1e-5
    # without bias, without bias gradient: the same bits elsewhere
    y2, dx2, dw2 = torch.empty_like(y), torch.empty_like(dx), torch.empty_like(dwt)
    L.lamp_convtr3d(x, wt, y2, bias=torch.zeros_like(b))
    y3 = torch.empty_like(y)
    L.lamp_convtr3d(x, wt, y3)
    assert torch.equal(y2, y3)
    L.lamp_convtr3d_bwd(x, wt, dy, dx=dx2, dwt=dw2)
    assert torch.equal(dx, dx2) and rel(dw2, r[2]) <= 1e-5
    # without the data gradient: the weight gradient alone
    dw4, db4 = torch.empty_like(dwt), torch.empty_like(db)
    L.lamp_convtr3d_bwd(x, wt, dy, dwt=dw4, dbias=db4)
    assert rel(dw4, r[2]) <= 1e-5 and rel(db4, r[3]) <= 1e-5


# more row blocks than workgroups are resident: 258 of 128 inputs, 513 of 16
@pytest.mark.parametrize("ci,co", [(128, 8256), (16, 16416)])
def test_convtr_fwd_many_outputs(L, ci, co):
    g = torch.Generator(device="cuda").manual_seed(co)
    x = torch.randn((1, 1, 2, 3, ci), generator=g, device="cuda").to(BF)
    wt = (torch.randn((ci, 2, 2, 2, co), generator=g, device="cuda") * ci ** -0.5).to(BF)
    b = torch.randn((co,), generator=g, device="cuda")
    y = torch.full((1, 2, 4, 6, co), 7.0, device="cuda").to(BF)
    L.lamp_convtr3d(x, wt, y, bias=b)
    r = (x.double().reshape(-1, ci) @ wt.double().reshape(ci, 8 * co)).reshape(1, 1, 2, 3, 2, 2, 2, co)
    r = r.permute(0, 1, 4, 2, 5, 3, 6, 7).reshape(y.shape) + b.double()
    assert rel(y, r) <= 2.0 ** -8   # one rounding to bf16


def cols64(dy, n, d, h, w):
    """dy as [voxels][8 * co], in chunks of 4096 voxels."""
    co = dy.shape[4]
    c = dy.reshape(n, d, 2, h, 2, w, 2, co).permute(0, 1, 3, 5, 2, 4, 6, 7).reshape(-1, 8 * co)
    out = torch.zeros((-(-len(c) // 4096) * 4096, 8 * co), dtype=torch.float64, device="cuda")
    out[:len(c)] = c
    return out.view(-1, 4096, 8 * co)


# Walks of the forward kernel over three groups of 32 voxels and more for every wave (512 workgroups of 8 waves up to 64 inputs, 256 by
# two row blocks with 128), with a ragged end; of the one-pass backward over nine chunks of 64 and more for every workgroup, so that all
# three stages are written over and, at 64 -> 32, chains of four chunks end twice.
@pytest.mark.parametrize("shape,co", [((1, 70, 64, 61, 16), 8), ((1, 67, 66, 67, 32), 16), ((1, 66, 64, 65, 64), 32), ((1, 53, 53, 54, 32), 32),
                                      ((1, 53, 53, 54, 64), 16), ((1, 45, 43, 41, 128), 64)], ids=str)
def test_convtr_long_walks(L, shape, co):
    g = torch.Generator(device="cuda").manual_seed(shape[4] + co)
    n, d, h, w, ci = shape
    x = torch.relu(torch.randn(shape, generator=g, device="cuda")).to(BF)
    dy = torch.randn((n, 2 * d, 2 * h, 2 * w, co), generator=g, device="cuda").to(BF)
    wt = (torch.randn((ci, 2, 2, 2, co), generator=g, device="cuda") * (2.0 / (8 * ci)) ** 0.5).to(BF)
    b = torch.randn((co,), generator=g, device="cuda")
    y, dx = torch.full_like(dy, 7.0), torch.full_like(x, 7.0)
    dw, db = torch.empty(wt.shape, device="cuda"), torch.empty((co,), device="cuda")
    L.lamp_convtr3d(x, wt, y, bias=b)
    L.lamp_convtr3d_bwd(x, wt, dy, dx=dx, dwt=dw, dbias=db)
    w64 = wt.double().reshape(ci, 8 * co)
    r = (x.double().reshape(-1, ci) @ w64).reshape(n, d, h, w, 2, 2, 2, co).permute(0, 1, 4, 2, 5, 3, 6, 7).reshape(y.shape) + b.double()
    assert rel(y, r) <= 2.0 ** -8   # one rounding to bf16
    del r
    c = cols64(dy, n, d, h, w)
    v = n * d * h * w
    xs = torch.zeros((c.shape[0] * 4096, ci), dtype=torch.float64, device="cuda")
    xs[:v] = x.reshape(-1, ci)
    assert rel(dx, (c.reshape(-1, 8 * co)[:v] @ w64.t().contiguous()).reshape(shape)) <= 2.0 ** -8
    rw = torch.bmm(xs.view(-1, 4096, ci).transpose(1, 2).contiguous(), c).sum(0).reshape(wt.shape)
    if ci > 64 or ci < 32:
        assert rel(dw, rw) <= 1e-6
        return
    # a chain of l additions carries 2^-24 / sqrt(3) * sqrt(l / 2): four products of 16 voxels a chunk, added in fp64 (64 -> 32: chains of
    # four chunks, up to three of them to a walk in fp32); a partial and the result rounded once each, as much as two additions.  Bias:
    # single products and the result (its partials are two floats)
    u = 2.0 ** -24 / math.sqrt(3.0)
    assert rel(dw, rw) <= u * math.sqrt(((16 + 3 if (ci, co) == (64, 32) else 4) + 4) / 2.0)
    assert rel(db, c.reshape(-1, 8, co).sum((0, 1))) <= u * math.sqrt((1 + 2) / 2.0)
