"""Transposed convolution on the bf16 kernels that walk groups and chunks of voxels: remainders of groups, chunks and walks, every weight
depth, channel slices, accumulation and missing outputs, against 64-bit torch."""
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


# 1, 31, 33 voxels and walks that end inside a group or chunk; 17000 voxels: more chunks than workgroups; weights off 16 bytes and 48
# input channels take the older kernels; 2 x 5 x 6 x 7 x 256 the unit-at-a-time kernel and the data gradient whose waves share a group
@pytest.mark.parametrize("shape,co,extra,woff", [((1, 1, 1, 1, 64), 32, 0, 0), ((1, 1, 1, 31, 64), 32, 8, 0), ((1, 3, 1, 11, 64), 32, 0, 0), ((2, 5, 7, 13, 64), 32, 0, 0),
                                                 ((1, 20, 25, 34, 64), 32, 0, 0), ((1, 3, 5, 7, 16), 8, 0, 0), ((2, 4, 5, 9, 32), 16, 8, 0),
                                                 ((1, 5, 6, 7, 128), 64, 0, 0), ((1, 3, 4, 5, 32), 24, 0, 0), ((1, 3, 4, 11, 16), 40, 8, 0),
                                                 ((1, 4, 5, 6, 64), 32, 0, 1), ((1, 4, 5, 6, 48), 32, 0, 0), ((2, 5, 6, 7, 256), 128, 0, 0),
                                                 ((2, 3, 3, 3, 64), 64, 0, 0)], ids=str)
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
