"""InstanceNorm + ReLU + max-pool row by row, and the windows of a volume in 16-byte pieces."""
import pytest
import torch

import lamp_synth as S
from gpu_chain import Chain
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu
BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


# base channels 8 to 256 are 1 to 32 channel vectors (rows), 24 and 48 no power of two (pooled voxels); rows that end within a block
# and within a wave, several samples
@pytest.mark.parametrize("affine", [False, True])
@pytest.mark.parametrize("base,shape", [(8, (1, 2, 2, 4)), (8, (3, 4, 6, 10)), (16, (2, 6, 4, 18)), (24, (1, 4, 6, 10)), (32, (2, 4, 6, 34)),
                                        (48, (1, 4, 4, 6)), (64, (1, 6, 2, 14)), (128, (2, 2, 4, 6)), (256, (1, 2, 2, 10))], ids=str)
def test_pool_rows(L, base, shape, affine):
    p = S.unet_params(S.streams(base + sum(shape), 1)[0], 2, base, 1, 3, affine, test_mode=True)
    dev = [to_dev(v, F32 if k.endswith((".b", ".gamma", ".beta")) else BF) for k, v in p.items()]
    x = to_dev(S.normal(S.streams(base, 2)[1], (*shape, 1)), BF)
    n, d, h, w = shape
    ud = L.unet_desc(2, base, 1, 3, *shape, BF, affine=affine)
    ws = torch.empty(L.lamp_unet_stage_workspace_bytes(ud, 1, 1), dtype=torch.uint8, device=DEV)
    pooled = torch.full((n, d // 2, h // 2, w // 2, base), float("nan"), dtype=BF, device=DEV)
    skip = torch.full((*shape, base), float("nan"), dtype=BF, device=DEV)
    L.lamp_unet_stage_fwd(ud, 1, 1, dev[:next(i for i, k in enumerate(p) if k.startswith("enc2"))], x, pooled, [skip], ws)
    ch = Chain(L, 2, base, 1, 3, affine, BF, list(p), dev, verify=False)
    ch.forward(x)   # the norm and the pooling as passes of their own: the same arithmetic, so the same bits
    assert torch.equal(skip, ch.enc[1][1]["y"]) and torch.equal(pooled, ch.pooled[1])


# 16-byte pieces: rows of 16 bytes' multiples, the last window moved in by a multiple of them; elements: width, window or stride are not
@pytest.mark.parametrize("dtype,ch,P,dims,overlap", [(BF, 1, 16, (16, 20, 40), 0.5), (BF, 2, 12, (13, 12, 20), 1 / 3), (F32, 1, 12, (12, 13, 20), 1 / 3),
                                                     (F32, 2, 8, (9, 8, 22), 0.25), (BF, 1, 16, (16, 17, 41), 0.5), (BF, 1, 12, (12, 12, 24), 0.5),
                                                     (F32, 1, 8, (8, 8, 20), 0.25), (F32, 3, 4, (5, 6, 12), 0.5), (BF, 3, 8, (8, 9, 16), 0.25)], ids=str)
def test_gather(L, dtype, ch, P, dims, overlap):
    step = round(P * (1 - overlap))
    ax = [sorted({min(i, s - P) for i in range(0, s - P + step, step)}) for s in dims]
    wins = [(i, j, k) for i in ax[0] for j in ax[1] for k in ax[2]]
    assert len(wins) == L.lamp_sliding_window_count(*dims, P, overlap)
    g = torch.Generator(device=DEV).manual_seed(P * ch + sum(dims))
    ud = L.unet_desc(2, 8, ch, 3, len(wins), P, P, P, dtype)
    p = S.unet_params(S.streams(P, 1)[0], 2, 8, ch, 3, False, test_mode=True)
    params = [to_dev(v, F32 if k.endswith(".b") else dtype) for k, v in p.items()]
    vol = torch.randn((1, *dims, ch), generator=g, device=DEV).to(dtype)
    out = torch.full((1, *dims, 3), float("nan"), device=DEV)
    L.lamp_sliding_window_fwd(ud, params, vol, out, overlap=overlap)
    logits = torch.empty((len(wins), P, P, P, 3), device=DEV)
    L.lamp_unet_fwd(ud, params, torch.stack([vol[0, i:i + P, j:j + P, k:k + P] for i, j, k in wins]), logits)
    e = torch.exp(-(torch.arange(P, dtype=torch.float64, device=DEV) - (P - 1) / 2.0) ** 2 / (2.0 * (0.125 * P) ** 2))
    w = e[:, None, None, None] * e[None, :, None, None] * e[None, None, :, None]
    num, den = torch.zeros((*dims, 3), dtype=torch.float64, device=DEV), torch.zeros((*dims, 1), dtype=torch.float64, device=DEV)
    cover = torch.zeros(dims, device=DEV)
    for q, (i, j, k) in enumerate(wins):
        num[i:i + P, j:j + P, k:k + P] += w * logits[q].double()
        den[i:i + P, j:j + P, k:k + P] += w
        cover[i:i + P, j:j + P, k:k + P] += 1
    ref = num / den
    # a weight carries the rounding of its exponent (up to 42 in size) and of expf, each window's term and sum a few more
    assert ((out[0].double() - ref).abs() <= 2.0 ** -24 * 60 * cover.max() * ref.abs().clamp_min(ref.abs().mean())).all()
