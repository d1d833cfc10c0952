"""Gaussian blend of sliding windows against the windows' own logits in 64 bits: one, two and four pieces of a volume row to a thread,
pieces of two floats (even class counts) and of one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def starts(size, patch, step):
    s = [0]
    while s[-1] + patch < size:
        s.append(min(s[-1] + step, size - patch))
    return s


# row of the volume in pieces: 16*4/2 = 32 and 16*3 (one a thread), 150*4/2 = 300 and 100*3 (two), 300*4/2 = 600, 180*3 = 540 and
# 1100*1 (four, the last over two blocks)
@pytest.mark.parametrize("classes,dims", [(4, (16, 17, 16)), (3, (17, 16, 16)), (4, (16, 16, 150)), (3, (16, 20, 100)), (4, (16, 16, 300)),
                                          (3, (16, 17, 180)), (1, (16, 16, 1100))], ids=str)
def test_blend(L, classes, dims):
    P, dev = 16, "cuda"
    g = torch.Generator(device=dev).manual_seed(classes * 1000 + dims[2])
    ax = [starts(s, P, 12) for s in dims]
    wins = [(i, j, k) for i in ax[0] for j in ax[1] for k in ax[2]]
    ud = L.unet_desc(2, 8, 1, classes, len(wins), P, P, P, torch.float32)
    params = [torch.randn(L.lamp_unet_param_numel(ud, i), generator=g, device=dev) * 0.1 for i in range(L.lamp_unet_param_count(ud))]
    vol = torch.randn((1, *dims, 1), generator=g, device=dev)
    out = torch.full((1, *dims, classes), float("nan"), device=dev)
    L.lamp_sliding_window_fwd(ud, params, vol, out)
    x = torch.stack([vol[0, i:i + P, j:j + P, k:k + P] for i, j, k in wins])
    logits = torch.empty((len(wins), P, P, P, classes), device=dev)
    L.lamp_unet_fwd(ud, params, x, logits)
    e = torch.exp(-(torch.arange(P, dtype=torch.float64, device=dev) - (P - 1) / 2.0) ** 2 / (2.0 * (0.125 * P) ** 2))
    w = e[:, None, None, None] * e[None, :, None, None] * e[None, None, :, None]
    num = torch.zeros((*dims, classes), dtype=torch.float64, device=dev)
    den = torch.zeros((*dims, 1), dtype=torch.float64, device=dev)
    for q, (i, j, k) in enumerate(wins):
        num[i:i + P, j:j + P, k:k + P] += w * logits[q].double()
        den[i:i + P, j:j + P, k:k + P] += w
    # at most eight windows cover a voxel; a weight carries the rounding of its exponent (up to 42 in size) and of expf, the rest a few more
    ref = num / den
    assert ((out[0].double() - ref).abs() <= 2.0 ** -24 * 60 * 8 * ref.abs().clamp_min(ref.abs().mean())).all()
