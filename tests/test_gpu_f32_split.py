"""fp32 convolutions with operands in bf16 pieces, at the edges of their tiles: every tile and block of outputs, ragged volumes and channel
counts, channel slices, one and several tiles a workgroup, against 64-bit torch; values at the ends of the fp32 range."""
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def shifted(x, t):
    D, H, W = x.shape[1:4]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
    return xp[:, t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[4])


def conv(x, w27):   # w27 [co][27][ci]
    return sum(shifted(x, t) @ w27[:, t].t() for t in range(27)).reshape(*x.shape[:4], -1)


def sliced(t, extra):
    buf = torch.full((*t.shape[:4], t.shape[4] + extra), float("nan"), device="cuda")
    buf[..., :t.shape[4]] = t
    return buf[..., :t.shape[4]]


def rel(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


# An instruction rounds its sum of 32 products a few times, two units each at most: chains of 27 co / 32 (weight gradient: 128, and as many
# sums of them again) such roundings of random sign, four units, and the rounding of the result.
@pytest.mark.parametrize("shape,co,extra", [
    ((1, 37, 35, 41, 8), 8, 0), ((2, 49, 31, 33, 4), 8, 4), ((1, 36, 40, 44, 16), 16, 0), ((2, 32, 25, 23, 12), 16, 8),
    ((1, 35, 36, 37, 24), 32, 0), ((1, 13, 11, 17, 20), 24, 0), ((1, 19, 23, 29, 48), 32, 4), ((1, 50, 40, 33, 32), 32, 0),
    ((1, 9, 7, 65, 96), 40, 0), ((3, 9, 10, 12, 64), 64, 0), ((1, 12, 9, 11, 72), 128, 0), ((1, 3, 64, 65, 8), 24, 0), ((1, 70, 29, 5, 24), 8, 0),
    ((2, 49, 3, 50, 48), 16, 12), ((1, 100, 61, 55, 16), 8, 0), ((1, 17, 16, 16, 32), 256, 0), ((1, 8, 8, 8, 32), 32, 0), ((1, 1, 2, 3, 8), 24, 0),
    ((1, 46, 47, 41, 8), 40, 0), ((2, 40, 70, 75, 8), 8, 0)], ids=str)
def test_f32_split(L, shape, co, extra):
    g = torch.Generator(device="cuda").manual_seed(sum(shape) + co)
    ci = shape[4]
    x = sliced(torch.randn(shape, generator=g, device="cuda"), extra)
    dz = sliced(torch.randn((*shape[:4], co), generator=g, device="cuda"), extra)
    w = torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * (2.0 / (27 * ci)) ** 0.5
    dx, dw = sliced(torch.zeros_like(x), extra), torch.randn(w.shape, generator=g, device="cuda")
    dw0 = dw.double()
    L.lamp_conv3d_dgrad(dz, w, dx)
    L.lamp_conv3d_wgrad(x, dz, dw, beta=1.0)
    dwr = torch.stack([dz.double().reshape(-1, co).t() @ shifted(x, t) for t in range(27)], 1).reshape(w.shape) + dw0
    assert rel(dx, conv(dz, w.double().reshape(co, 27, ci).flip(1).permute(2, 1, 0))) <= 4 * U * (27 * co / 32) ** 0.5 + U
    assert rel(dw, dwr) <= 4 * U * 256 ** 0.5 + U
    assert torch.isnan(dx.as_strided((*shape[:4], ci + extra), dx.stride())[..., ci:]).all()   # nothing beside the slice


# A gradient whose many small values are of one sign, over a non-negative input: no product may be cut off to one side, which would add up
# over the voxels.  As far from 64 bits as fp32 products in chains of 128 voxels (1.8e-7 in each of these sizes) at most; measured 5e-8 to 8e-8.
@pytest.mark.parametrize("shape,co", [((1, 41, 56, 47, 32), 32), ((2, 64, 48, 80, 8), 8), ((2, 64, 48, 80, 16), 16), ((1, 53, 64, 29, 48), 64)], ids=str)
@pytest.mark.parametrize("spread", [0.0, 1.0])
def test_weight_gradient_of_one_sided_gradients(L, shape, co, spread):
    g = torch.Generator(device="cuda").manual_seed(co)
    r = lambda s: torch.randn(s, generator=g, device="cuda")
    z = r((*shape[:4], co))
    up = r(z.shape) * (z > 0)
    dz = up - up.mean((1, 2, 3), keepdim=True) - z * (up * z).mean((1, 2, 3), keepdim=True)
    x, dz = torch.relu(r(shape)) * torch.exp(spread * r((shape[4],))), dz * torch.exp(spread * r((co,)))
    dw = torch.empty((co, 3, 3, 3, shape[4]), device="cuda")
    L.lamp_conv3d_wgrad(x, dz, dw)
    assert rel(dw, torch.stack([dz.double().reshape(-1, co).t() @ shifted(x, t) for t in range(27)], 1).reshape(dw.shape)) <= 1.8e-7


@pytest.mark.parametrize("shape,co,c_norm", [((1, 37, 35, 41, 8), 8, 8), ((1, 36, 40, 44, 16), 16, 12), ((2, 34, 35, 17, 32), 40, 32)], ids=str)
def test_weight_gradient_normalises_on_load(L, shape, co, c_norm):
    """The bits of the weight gradient of the normalised tensor."""
    g = torch.Generator(device="cuda").manual_seed(co)
    r = lambda s: torch.randn(s, generator=g, device="cuda")
    n, c = shape[0], shape[4]
    x, dz = r(shape), r((*shape[:4], co))
    nm = dict(mean_rstd=torch.stack([r((n, c_norm)) * 0.1, r((n, c_norm)).abs() + 0.5], -1).contiguous(), gamma=r((c_norm,)), beta=r((c_norm,)))
    y = x.clone()
    L.lamp_inorm_relu(x[..., :c_norm].contiguous(), y[..., :c_norm], nm["mean_rstd"], gamma=nm["gamma"], beta=nm["beta"], stats_given=True)
    dw, dwn = (torch.empty((co, 3, 3, 3, c), device="cuda") for _ in range(2))
    L.lamp_conv3d_wgrad(y, dz, dw)
    L.lamp_conv3d_wgrad(x, dz, dwn, xnorm=dict(nm, c_norm=c_norm, relu=1))
    assert torch.equal(dw, dwn)


@pytest.mark.parametrize("ci,co", [(8, 8), (16, 16), (40, 32)], ids=str)
def test_ends_of_the_range(L, ci, co):
    """Infinities, NaN and the largest values come out of the data gradient as with fp32 products; powers of two move no bit.  The weight
    gradient of an output channel that holds one is not finite where the sum is not, and the other channels are as without it."""
    g = torch.Generator(device="cuda").manual_seed(ci)
    shape = (1, 37, 36, 41, co)
    dz = torch.randn(shape, generator=g, device="cuda")
    w = torch.randn((co, 3, 3, 3, ci), generator=g, device="cuda") * 0.1
    x = torch.randn((*shape[:4], ci), generator=g, device="cuda")
    dx0, dx = (torch.empty((*shape[:4], ci), device="cuda") for _ in range(2))
    dw0, dw = (torch.empty_like(w) for _ in range(2))
    L.lamp_conv3d_dgrad(dz, w, dx0)
    L.lamp_conv3d_wgrad(x, dz, dw0)
    for s in (2.0 ** -90, 2.0 ** 60):
        L.lamp_conv3d_dgrad(dz * s, w, dx)
        L.lamp_conv3d_wgrad(x, dz * s, dw)
        assert torch.equal(dx, dx0 * s) and torch.equal(dw, dw0 * s)
    L.lamp_conv3d_wgrad(x, dz * 2.0 ** 115, dw)   # past the grids' range
    assert rel(dw * 2.0 ** -115, dw0.double()) <= 1e-6
    dz[0, 5, 6, 7, 1], dz[0, 20, 20, 20, 0], dz[0, 30, 5, 9, co - 1] = float("inf"), float("-inf"), float("nan")
    dz[0, 10, 30, 30, 2] = 3.4e38   # rounds to an infinity in bf16
    w[2] = 0.01
    L.lamp_conv3d_dgrad(dz, w, dx)
    # data gradient: the conv with taps reversed and channels exchanged
    dr = torch.nn.functional.conv3d(dz.cpu().permute(0, 4, 1, 2, 3), w.cpu().permute(4, 0, 1, 2, 3).flip(2, 3, 4), padding=1).permute(0, 2, 3, 4, 1).cuda()
    assert torch.equal(torch.isnan(dx), torch.isnan(dr)) and torch.equal(torch.isinf(dx), torch.isinf(dr))
    inf, fin = torch.isinf(dr), torch.isfinite(dr)
    assert inf.sum().item() == 2 * 27 * ci and torch.equal(dx[inf], dr[inf])
    big = fin & (dr.abs() > 1e30)
    assert big.sum().item() == 27 * ci and ((dx[big] - dr[big]) / dr[big]).abs().max().item() <= 4 * U
    rest = fin & ~big
    assert (dx[rest] - dr[rest]).abs().max().item() <= 1e-4
    L.lamp_conv3d_wgrad(x, dz, dw)
    bad, good = [0, 1, co - 1], list(range(3, co - 1))   # (channel 2: 3.4e38 times an input above 1 overflows in any arithmetic)
    assert not torch.isfinite(dw[bad]).any() and rel(dw[good], dw0[good].double()) <= 4 * U * 16


CHILD = """
import sys
import torch
sys.path.insert(0, %r)
import paper_2006_12575_amd as L
L.lib()
torch.manual_seed(5)
x, dz = (torch.randn((1, 30, 31, 33, 32), device="cuda") for _ in range(2))
w, dx, dw = torch.randn((32, 3, 3, 3, 32), device="cuda"), torch.empty_like(x), torch.empty((32, 3, 3, 3, 32), device="cuda")
ws = torch.empty(1 << 27, dtype=torch.uint8, device="cuda")

def call():
    L.lamp_conv3d_dgrad(dz, w, dx, ws=ws)
    L.lamp_conv3d_wgrad(x, dz, dw, ws=ws)
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    call()
got = []
for _ in range(3):
    dx.fill_(float("nan")), dw.fill_(float("nan"))
    g.replay()
    torch.cuda.synchronize()
    got.append((dx.clone(), dw.clone()))
call()
torch.cuda.synchronize()
assert all(torch.equal(a, dx) and torch.equal(b, dw) for a, b in got) and torch.isfinite(dx).all() and torch.isfinite(dw).all()
print("replays equal")
"""


def test_first_call_in_a_capture():
    import subprocess
    import sys

    import conftest
    r = subprocess.run([sys.executable, "-c", CHILD % conftest.ROOT], capture_output=True, text=True, timeout=90)
    assert r.returncode == 0 and "replays equal" in r.stdout, r.stderr[-2000:]
