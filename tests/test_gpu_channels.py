"""Channel counts that do not fill the matrix-core kernels' chunks of 16 and blocks of 32: every conv pass against the
CPU oracle, on both tile depths, both block widths, with bias, statistics, channel slices and accumulation."""
import numpy as np
import pytest
import torch

import lamp_synth as S
import oracle as O
from gpu_util import DEV, as64, check, to_dev

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def conv_passes(L, dtype, shape, seed, wgrad_tol, dgrad=True):
    """Forward (bias, statistics, into a slice of a wider buffer), data gradient, weight gradient (from slices, beta 0 and
    1) of one shape; inputs sit in wider buffers whose other channels are NaN, so that a read past the slice shows."""
    N, D, H, W, Ci, Co = shape
    r = rng(seed + sum(shape))
    nan = float("nan")

    def sliced(c, ref=None):   # c channels behind 8 others, 8 more behind them
        buf = torch.full((N, D, H, W, c + 16), nan, dtype=dtype, device=DEV)
        if ref is not None:
            buf[..., 8:8 + c] = to_dev(ref, dtype)
        return buf, buf[..., 8:8 + c]

    _, x = sliced(Ci, S.normal(r, (N, D, H, W, Ci)) + 0.25)
    w = to_dev(S.kaiming_conv(r, Co, Ci), dtype)
    b = to_dev(S.normal(r, (Co,), 0.1), F32)
    zbuf, z = sliced(Co)
    stats = torch.full((N, Co, 2), nan, dtype=F32, device=DEV)
    L.lamp_conv3d_fwd(x, w, z, bias=b, stats_out=stats)
    check(as64(z), O.conv3d_fwd(as64(x), as64(w), as64(b)), dtype, "conv fwd")
    assert torch.isnan(zbuf[..., :8]).all() and torch.isnan(zbuf[..., 8 + Co:]).all(), "wrote outside the channel slice"
    _, st_ref = O.inorm_relu(as64(z))
    check(as64(stats)[..., 0], st_ref[..., 0], F32, "stats mean", tol=1e-4)
    if D * H * W > 1:
        np.testing.assert_allclose(as64(stats)[..., 1], st_ref[..., 1], rtol=2e-4)
    z2 = torch.empty((N, D, H, W, Co), dtype=dtype, device=DEV)
    L.lamp_conv3d_fwd(x.contiguous(), w, z2, bias=b)
    assert torch.equal(z2, z)
    _, dz = sliced(Co, S.normal(r, (N, D, H, W, Co)))
    if dgrad:
        dxbuf, dx = sliced(Ci)
        L.lamp_conv3d_dgrad(dz, w, dx)
        check(as64(dx), O.conv3d_dgrad(as64(dz), as64(w)), dtype, "conv dgrad")
        assert torch.isnan(dxbuf[..., :8]).all() and torch.isnan(dxbuf[..., 8 + Ci:]).all(), "wrote outside the channel slice"
    dw = torch.full((Co, 3, 3, 3, Ci), nan, dtype=F32, device=DEV)
    db = torch.full((Co,), nan, dtype=F32, device=DEV)
    L.lamp_conv3d_wgrad(x, dz, dw, dbias=db)
    dw_ref, db_ref = O.conv3d_wgrad(as64(x), as64(dz), want_db=True)
    check(as64(dw), dw_ref, dtype, "conv wgrad", tol=wgrad_tol)
    check(as64(db), db_ref, dtype, "conv dbias", tol=1e-4)
    L.lamp_conv3d_wgrad(x, dz, dw, dbias=db, beta=1.0)
    check(as64(dw), 2 * dw_ref, dtype, "conv wgrad beta=1", tol=wgrad_tol)


# bf16 tolerances: one rounding to storage (1e-2 as everywhere, 2e-3 for the fp32 weight gradient of bf16 inputs)
@pytest.mark.parametrize("shape", [
    (1, 9, 10, 18, 8, 8),        # one half chunk, a quarter of a block
    (2, 5, 9, 17, 24, 40),       # half a last chunk; 40 = 64-wide block with 24 channels missing
    (1, 6, 17, 20, 48, 96),      # whole chunks, three 32-wide blocks; data gradient with 48 outputs
    (2, 8, 8, 16, 16, 72),       # three blocks, the last with 8 channels
    (1, 3, 5, 7, 104, 120),
    (6, 4, 4, 4, 24, 40),        # batch of tiny volumes in the packed layout
    (1, 260, 3, 5, 8, 16),       # more slices than the missing-channel mark of the weight gradient's copies
    (1, 64, 64, 64, 24, 24),     # 8-deep tile, 32-wide block
    (1, 64, 64, 60, 16, 48),     # 8-deep tile, 64-wide block
    (2, 64, 96, 112, 8, 24),     # statistics partials per walk
    (1, 1, 1, 1, 40, 8),
], ids=lambda s: "x".join(map(str, s)))
def test_conv3d_ragged_channels_bf16(L, shape):
    conv_passes(L, BF, shape, 2100, 2e-3)


@pytest.mark.parametrize("shape", [(1, 6, 9, 33, 2, 16), (2, 5, 6, 7, 3, 24), (1, 7, 9, 16, 12, 64), (1, 5, 6, 9, 4, 32),
                                   (5, 4, 4, 4, 20, 32), (1, 4, 5, 6, 1, 40),
                                   # two to four channels forward: 256-voxel tiles with one and two blocks of 16 outputs, then 128 and 64
                                   (1, 41, 40, 44, 2, 16), (1, 41, 40, 44, 3, 40), (1, 33, 32, 34, 2, 24), (1, 20, 28, 36, 4, 24)],
                         ids=lambda s: "x".join(map(str, s)))
def test_conv3d_narrow_input_bf16(L, shape):
    """Input channels that fill no 16-byte piece: padded with zero channels in the workspace for the gradients, on the fp32 matrix
    instruction (two to four) or the scalar kernels forward."""
    conv_passes(L, BF, shape, 2200, 2e-3)


@pytest.mark.parametrize("shape", [(8, 4, 4, 4, 8, 8), (40, 6, 6, 6, 8, 1), (75, 7, 7, 7, 8, 8), (100, 7, 7, 7, 8, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_conv3d_dgrad_tiny_batch_bf16(L, shape):
    """8 channels on batches of tiny volumes: up to 32768 voxels the scalar kernel, above the matrix-core one on the packed batch."""
    N, D, H, W, Ci, Co = shape
    r = rng(2250 + N)
    dz, w = to_dev(S.normal(r, (N, D, H, W, Co)), BF), to_dev(S.kaiming_conv(r, Co, Ci), BF)
    dx = torch.full((N, D, H, W, Ci), float("nan"), dtype=BF, device=DEV)
    L.lamp_conv3d_dgrad(dz, w, dx)
    check(as64(dx), O.conv3d_dgrad(as64(dz), as64(w)), BF, "conv dgrad")


def test_conv3d_ragged_channels_unaligned_weights(L):
    """Channel counts outside 16 / 32 take weights at any alignment (the scalar kernels read them)."""
    r = rng(2300)
    x = to_dev(S.normal(r, (1, 4, 5, 9, 24)), BF)
    wh = to_dev(S.kaiming_conv(r, 40, 24), BF)
    flat = torch.empty(wh.numel() + 1, dtype=BF, device=DEV)
    flat[1:] = wh.reshape(-1)
    w = flat[1:].view(wh.shape)
    z = torch.empty((1, 4, 5, 9, 40), dtype=BF, device=DEV)
    L.lamp_conv3d_fwd(x, w, z)
    check(as64(z), O.conv3d_fwd(as64(x), as64(wh)), BF, "conv fwd")
    dx = torch.empty_like(x)
    L.lamp_conv3d_dgrad(z, w, dx)
    check(as64(dx), O.conv3d_dgrad(as64(z), as64(wh)), BF, "conv dgrad")


# fp32: a sum of K <= 27 * 80 products carries about sqrt(K) * 2^-24 = 3e-6 of its terms' scale; weight gradients sum over up to
# 70000 voxels (1.6e-5) in partials of at most a few thousand
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 1, 1, 1),
    (1, 5, 6, 7, 1, 8),          # 64-voxel tiles; channel chunks of 4: one, two, three, four channels
    (2, 5, 9, 17, 2, 17),        # one channel in the last block of 16
    (1, 6, 9, 33, 3, 33),
    (2, 3, 20, 12, 4, 16),
    (1, 7, 9, 10, 5, 24),        # chunks of 8 cut short
    (1, 8, 8, 8, 8, 8),
    (3, 4, 5, 6, 20, 40),
    (1, 9, 10, 11, 32, 16),      # chunks of 16
    (1, 4, 4, 4, 80, 72),
    (1, 33, 32, 34, 16, 16),     # 128-voxel tiles
    (1, 33, 32, 34, 8, 32),      # with blocks of 32 outputs; chunks of 8 and of 4
    (1, 33, 32, 34, 2, 24),
    (1, 33, 32, 34, 20, 8),      # the same in the data gradient
    (1, 41, 40, 44, 16, 24),     # 256-voxel tiles
    (1, 33, 32, 34, 8, 48),
    (2, 33, 40, 47, 2, 8),
    (1, 41, 40, 44, 9, 12),
    (1, 41, 40, 44, 3, 40),
    (1, 41, 40, 44, 24, 3),
    (1, 20, 28, 36, 2, 24),      # 64-voxel tiles with blocks of 32 outputs, forward and data gradient
    (1, 20, 28, 36, 32, 4),
    (1, 5, 6, 7, 3, 72),         # more than 64 output channels: 16-voxel waves, 4-byte and 16-byte loads
    (2, 4, 9, 11, 20, 100),
    (1, 33, 32, 34, 16, 128),    # 64-voxel waves
    (1, 33, 32, 34, 6, 130),
], ids=lambda s: "x".join(map(str, s)))
def test_conv3d_f32(L, shape):
    conv_passes(L, F32, shape, 2400, 1e-4)


def test_conv3d_f32_unaligned(L):
    """fp32 tensors and weights off 16 bytes, channel strides that are no multiple of 4; a partial normalise-on-load, forward and in
    the weight gradient."""
    r = rng(2500)
    N, D, H, W, Ci, Co = 2, 5, 6, 19, 16, 20

    def off(ref, extra):   # channels 1.. of a buffer with `extra` more channels
        buf = torch.full((*ref.shape[:-1], ref.shape[-1] + extra), float("nan"), dtype=F32, device=DEV)
        buf[..., 1:1 + ref.shape[-1]] = to_dev(ref, F32)
        return buf[..., 1:1 + ref.shape[-1]]

    x = off(S.normal(r, (N, D, H, W, Ci)), 3)
    dz = off(S.normal(r, (N, D, H, W, Co)), 2)
    wh = S.kaiming_conv(r, Co, Ci)
    flat = torch.empty(wh.size + 1, dtype=F32, device=DEV)
    flat[1:] = to_dev(wh, F32).reshape(-1)
    w = flat[1:].view(wh.shape)
    z = off(np.zeros((N, D, H, W, Co)), 2)
    L.lamp_conv3d_fwd(x, w, z)
    check(as64(z), O.conv3d_fwd(as64(x), as64(w)), F32, "conv fwd")
    dx = off(np.zeros((N, D, H, W, Ci)), 3)
    L.lamp_conv3d_dgrad(dz, w, dx)
    check(as64(dx), O.conv3d_dgrad(as64(dz), as64(w)), F32, "conv dgrad")
    dw = torch.empty(wh.shape, dtype=F32, device=DEV)
    L.lamp_conv3d_wgrad(x, dz, dw)
    check(as64(dw), O.conv3d_wgrad(as64(x), as64(dz))[0], F32, "conv wgrad")
    cn = 10
    st = torch.stack([to_dev(S.normal(r, (N, cn), 0.1), F32), to_dev(S.normal(r, (N, cn)), F32).abs() + 0.5], -1).contiguous()
    xh = as64(x).copy()
    m = as64(st)[:, None, None, None]
    xh[..., :cn] = np.maximum(0.0, (xh[..., :cn] - m[..., 0]) * m[..., 1])
    nm = dict(mean_rstd=st, c_norm=cn, relu=1)
    L.lamp_conv3d_fwd(x, w, z, xnorm=nm)
    check(as64(z), O.conv3d_fwd(xh, as64(w)), F32, "conv fwd, normalise-on-load")
    L.lamp_conv3d_wgrad(x, dz, dw, xnorm=nm)
    check(as64(dw), O.conv3d_wgrad(xh, as64(dz))[0], F32, "conv wgrad, normalise-on-load")


# the transposed conv: fp32 on both wave tilings and both channel-block widths, bf16 weight gradient with channels past its blocks;
# tolerances as for the 3x3x3 passes, the bias gradient sums up to 8 * 66000 values in fp32 partials of about a thousand
@pytest.mark.parametrize("shape", [
    (F32, 1, 1, 1, 1, 4, 4), (F32, 2, 3, 5, 7, 20, 12), (F32, 1, 6, 7, 9, 16, 8), (F32, 3, 5, 4, 6, 64, 36), (F32, 1, 33, 40, 50, 32, 16),
    (F32, 1, 41, 40, 41, 40, 4),
    (BF, 1, 3, 4, 5, 16, 8), (BF, 2, 5, 6, 7, 32, 16), (BF, 1, 9, 8, 11, 80, 40), (BF, 1, 33, 40, 50, 48, 24),
], ids=lambda s: "x".join(map(str, s)))
def test_convtr3d_channels(L, shape):
    dtype, N, D, H, W, Ci, Co = shape
    r = rng(2600 + sum(shape[1:]))
    nan = float("nan")

    def sliced(dims, c, ref=None):
        buf = torch.full((*dims, c + 16), nan, dtype=dtype, device=DEV)
        if ref is not None:
            buf[..., 8:8 + c] = to_dev(ref, dtype)
        return buf, buf[..., 8:8 + c]

    co, fi = (N, D, H, W), (N, 2 * D, 2 * H, 2 * W)
    _, x = sliced(co, Ci, S.normal(r, (*co, Ci)))
    wt = to_dev(S.kaiming_convtr(r, Ci, Co), dtype)
    b = to_dev(S.normal(r, (Co,), 0.1), F32)
    ybuf, y = sliced(fi, Co)
    L.lamp_convtr3d(x, wt, y, bias=b)
    check(as64(y), O.convtr3d_fwd(as64(x), as64(wt), as64(b)), dtype, "convtr fwd")
    assert torch.isnan(ybuf[..., :8]).all() and torch.isnan(ybuf[..., 8 + Co:]).all()
    _, dy = sliced(fi, Co, S.normal(r, (*fi, Co)) + 0.25)
    dxbuf, dx = sliced(co, Ci)
    dwt = torch.full(wt.shape, nan, dtype=F32, device=DEV)
    db = torch.full((Co,), nan, dtype=F32, device=DEV)
    L.lamp_convtr3d_bwd(x, wt, dy, dx=dx, dwt=dwt, dbias=db)
    dx_ref, dwt_ref, db_ref = O.convtr3d_bwd(as64(x), as64(wt), as64(dy))
    tol = 1e-4 if dtype == F32 else 2e-3
    check(as64(dx), dx_ref, dtype, "convtr dgrad")
    assert torch.isnan(dxbuf[..., :8]).all() and torch.isnan(dxbuf[..., 8 + Ci:]).all()
    check(as64(dwt), dwt_ref, dtype, "convtr wgrad", tol=tol)
    check(as64(db), db_ref, dtype, "convtr dbias", tol=1e-4)
    L.lamp_convtr3d_bwd(x, wt, dy, dwt=dwt, dbias=db, beta=1.0)
    check(as64(dwt), 2 * dwt_ref, dtype, "convtr wgrad beta=1", tol=tol)
    check(as64(db), 2 * db_ref, dtype, "convtr dbias beta=1", tol=1e-4)
