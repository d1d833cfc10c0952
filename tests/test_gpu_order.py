"""The order of the forward pass's sums: up to 64 outputs normalise-on-load gives the bits of the conv of the normalised tensor, and
the matrix instructions give the bits of fused multiply-adds taken one after the other."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def rand(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda shape, dtype=F32: torch.randn(shape, generator=g, device="cuda").to(dtype)


# fp32 with more than 64 outputs takes its sums in another order than without xnorm: the same to rounding, sums of up to 27 * 24
# products in either order
@pytest.mark.parametrize("dtype,shape,co,c_norm", [(F32, (2, 5, 6, 7, 16), 64, 16), (F32, (2, 5, 6, 7, 16), 72, 16), (F32, (1, 9, 10, 11, 24), 100, 8),
                                                   (F32, (2, 4, 9, 11, 7), 40, 5), (F32, (2, 33, 32, 17, 8), 48, 8), (F32, (2, 20, 28, 36, 4), 24, 4),
                                                   (BF, (2, 9, 8, 10, 2), 16, 2), (BF, (2, 20, 28, 36, 3), 24, 2), (BF, (1, 41, 40, 44, 4), 40, 4)],
                         ids=str)
def test_normalise_on_load_bits(L, dtype, shape, co, c_norm):
    r = rand(sum(shape) + co)
    n, c = shape[0], shape[4]
    x, w, b = r(shape, dtype), (r((co, 3, 3, 3, c)) * (2.0 / (27 * c)) ** 0.5).to(dtype), r((co,))
    st = torch.stack([r((n, c_norm)) * 0.1, r((n, c_norm)).abs() + 0.5], -1).contiguous()
    ga, be = r((c_norm,)), r((c_norm,))
    y = x.clone()
    L.lamp_inorm_relu(x[..., :c_norm].contiguous(), y[..., :c_norm], st, gamma=ga, beta=be, stats_given=True)
    z, zn = (torch.empty((*shape[:4], co), dtype=dtype, device="cuda") for _ in range(2))
    L.lamp_conv3d_fwd(y, w, z, bias=b)
    L.lamp_conv3d_fwd(x, w, zn, bias=b, xnorm=dict(mean_rstd=st, gamma=ga, beta=be, c_norm=c_norm, relu=1))
    if dtype == F32 and co > 64:
        assert ((z - zn).norm() / z.norm()).item() <= 2.0 ** -24 * (27 * 24) ** 0.5
    else:
        assert torch.equal(z, zn)


def fma_chain(x, w, v, co, order):
    """One output of the forward pass, as fused multiply-adds in `order` (list of (tap, channel))."""
    fmaf = ctypes.CDLL("libm.so.6").fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    n, d, h, ww = v
    D, H, W = x.shape[1:4]
    acc = 0.0
    for t, c in order:
        a, b, e = d + t // 9 - 1, h + t // 3 % 3 - 1, ww + t % 3 - 1
        if 0 <= a < D and 0 <= b < H and 0 <= e < W:
            acc = fmaf(float(x[n, a, b, e, c]), float(w[co, t, c]), acc)
    return np.float32(acc)


# up to 64 outputs: chunks of 8 channels, in a chunk the taps, in a tap the channels; above: taps, then channels
@pytest.mark.parametrize("shape,co", [((1, 5, 6, 7, 3), 8), ((2, 6, 5, 9, 20), 24), ((1, 9, 10, 11, 32), 40), ((1, 20, 28, 36, 16), 16),
                                      ((1, 4, 5, 6, 20), 72), ((1, 33, 32, 34, 8), 128)], ids=str)
def test_sums_are_chains_of_fused_multiply_adds(L, shape, co):
    r = rand(sum(shape) + co)
    c = shape[4]
    x, w = r(shape), r((co, 3, 3, 3, c)) * 0.2
    z = torch.empty((*shape[:4], co), device="cuda")
    L.lamp_conv3d_fwd(x, w, z)
    if co <= 64:
        order = [(t, k) for c0 in range(0, c, 8) for t in range(27) for k in range(c0, min(c0 + 8, c))]
    else:
        order = [(t, k) for t in range(27) for k in range(c)]
    xh, wh, zh = x.cpu().numpy(), w.reshape(co, 27, c).cpu().numpy(), z.cpu().numpy()
    pick = np.random.Generator(np.random.PCG64(7))
    for _ in range(60):
        v = tuple(int(pick.integers(0, s)) for s in shape[:4])
        k = int(pick.integers(0, co))
        ref = fma_chain(xh, wh, v, k, order)
        assert zh[v][k] == ref, (v, k, zh[v][k], ref)


@pytest.mark.parametrize("shape,co", [((2, 16, 20, 24, 2), 16), ((1, 41, 40, 44, 2), 16), ((1, 33, 40, 47, 3), 48), ((2, 7, 9, 11, 4), 8)], ids=str)
def test_narrow_bf16_input_equals_scalar_kernel(L, shape, co):
    """A z whose voxels do not start on 8 bytes is left to the scalar kernel: the same bits, statistics up to their last ones."""
    r = rand(sum(shape) + co)
    x, w = r(shape, BF), (r((co, 3, 3, 3, shape[4])) * 0.2).to(BF)
    z = torch.empty((*shape[:4], co), dtype=BF, device="cuda")
    odd = torch.empty((*shape[:4], co + 1), dtype=BF, device="cuda")[..., :co]
    st, so = (torch.empty((shape[0], co, 2), device="cuda") for _ in range(2))
    L.lamp_conv3d_fwd(x, w, z, stats_out=st)
    L.lamp_conv3d_fwd(x, w, odd, stats_out=so)
    assert torch.equal(z, odd)
    torch.testing.assert_close(st, so, rtol=1e-5, atol=1e-6)
