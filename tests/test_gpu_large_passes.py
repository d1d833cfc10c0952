"""Passes over more bytes than the memory-side cache holds take non-temporal accesses (and the max-pool backward another lane
mapping): a batch beyond the limit must give bit for bit what its samples give one by one below it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
LIMIT = 256 << 20


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def rand(gen, shape, dtype=BF):
    return torch.randn(shape, generator=gen, device="cuda").to(dtype)


@pytest.mark.parametrize("dtype,shape", [(BF, (4, 64, 96, 96, 64)), (BF, (5, 63, 97, 95, 48)), (F32, (4, 62, 66, 70, 56))],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s)[6:])
def test_norm_and_gate_batch_equals_samples(L, dtype, shape):
    g = torch.Generator(device="cuda").manual_seed(31)
    n, d, h, w, c = shape
    es = 2 if dtype == BF else 4
    assert 2 * n * d * h * w * c * es > LIMIT > 3 * d * h * w * c * es
    z, dy, res = (rand(g, shape, dtype) for _ in range(3))
    ga, be = rand(g, (c,), F32), rand(g, (c,), F32)
    st = torch.stack([rand(g, (n, c), F32) * 0.1, rand(g, (n, c), F32).abs() + 0.5], -1).contiguous()
    cr = c // 4
    w1, b1, w2, b2 = rand(g, (cr, c), F32), rand(g, (cr,), F32), rand(g, (c, cr), F32), rand(g, (c,), F32)

    def passes(z, dy, res, st):
        y, dz, ys, dzs = (torch.empty_like(z) for _ in range(4))
        L.lamp_inorm_relu(z, y, st, gamma=ga, beta=be, stats_given=True)
        L.lamp_inorm_relu_bwd(dy, z, st, dz, gamma=ga, beta=be)
        gate = torch.empty((z.shape[0], 4 * c + cr), dtype=F32, device="cuda")
        L.lamp_inorm_relu_se(z, st, w1, w2, ys, gate, b1=b1, b2=b2, gamma=ga, beta=be, residual=res)
        L.lamp_inorm_relu_se_bwd(dy, z, st, w1, w2, gate, dzs, gamma=ga, beta=be)
        return y, dz, ys, dzs

    whole = passes(z, dy, res, st)
    for i in range(n):
        for a, b in zip(whole, passes(z[i:i + 1], dy[i:i + 1], res[i:i + 1], st[i:i + 1].contiguous())):
            assert torch.equal(a[i:i + 1], b)


@pytest.mark.parametrize("dtype,shape", [(BF, (4, 64, 96, 96, 64)), (BF, (9, 62, 66, 74, 40)), (F32, (5, 46, 66, 70, 36))],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s)[6:])
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "add"])
def test_maxpool_bwd_batch_equals_samples(L, dtype, shape, skip):
    g = torch.Generator(device="cuda").manual_seed(32)
    n, d, h, w, c = shape
    es = 2 if dtype == BF else 4
    assert 2 * n * d * h * w * c * es > LIMIT > 2 * d * h * w * c * es
    x = torch.relu(rand(g, shape, dtype))   # ties among zeros: the first of a window gets the gradient
    add = rand(g, shape, dtype) if skip else None
    dy = rand(g, (n, d // 2, h // 2, w // 2, c), dtype)
    dx = torch.empty_like(x)
    L.lamp_maxpool2_bwd(x, dy, dx, add=add)
    for i in range(n):
        one = torch.empty_like(x[i:i + 1])
        L.lamp_maxpool2_bwd(x[i:i + 1], dy[i:i + 1], one, add=add[i:i + 1] if skip else None)
        assert torch.equal(dx[i:i + 1], one)


@pytest.mark.parametrize("shape", [(9, 64, 96, 96, 32), (5, 61, 95, 104, 64)], ids=lambda s: "x".join(map(str, s)))   # a sample starts on 16 bytes
def test_first_layer_batch_equals_samples(L, shape):
    g = torch.Generator(device="cuda").manual_seed(33)
    n, d, h, w, c = shape
    assert 2 * n * d * h * w * c > LIMIT > 2 * d * h * w * c
    x, wt = rand(g, (n, d, h, w, 1)), rand(g, (c, 3, 3, 3, 1))
    z = torch.empty(shape, dtype=BF, device="cuda")
    L.lamp_conv3d_fwd(x, wt, z)
    for i in range(n):
        one = torch.empty((1, d, h, w, c), dtype=BF, device="cuda")
        L.lamp_conv3d_fwd(x[i:i + 1], wt, one)
        assert torch.equal(z[i:i + 1], one)
