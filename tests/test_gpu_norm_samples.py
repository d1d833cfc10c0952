"""Norm and gate backward over one to many samples, with both, one or none of the affine parameters' gradients wanted, on small tensors
(whose apply pass folds the partial sums itself) and larger ones, against 64-bit torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


def rel(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


# up to 512 partials x channels: folded by the apply pass, unless several samples and a gradient; C = 300 and 520: channels one by one
@pytest.mark.parametrize("wanted", ["both", "gamma", "beta", "none"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 4, 4, 4, 256), (3, 4, 4, 4, 256), (2, 3, 4, 5, 64), (75, 4, 4, 4, 64), (9, 5, 6, 7, 16), (8, 4, 4, 4, 300),
                                   (17, 3, 3, 5, 520), (2, 12, 11, 13, 128), (3, 2, 3, 4, 2056)], ids=str)
def test_inorm_bwd_samples(L, shape, dtype, wanted):
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    n, c = shape[0], shape[4]
    z, dy = (torch.randn(shape, generator=g, device="cuda").to(dtype) for _ in range(2))
    z64 = z.double()
    m = z64.mean((1, 2, 3))
    st = torch.stack([m, torch.rsqrt(z64.var((1, 2, 3), unbiased=False) + 1e-5)], -1).float().contiguous()
    ga, be = (torch.rand((c,), generator=g, device="cuda") + o for o in (0.5, -0.5))
    dga = torch.ones((c,), device="cuda") if wanted in ("both", "gamma") else None
    dbe = torch.full((c,), 2.0, device="cuda") if wanted in ("both", "beta") else None
    dz = torch.empty_like(z)
    L.lamp_inorm_relu_bwd(dy, z, st, dz, gamma=ga, beta=be, dgamma=dga, dbeta=dbe, beta_acc=1.0)
    z64.requires_grad_(True)
    p = [ga.double().requires_grad_(True), be.double().requires_grad_(True)]
    d = z64 - z64.mean((1, 2, 3), keepdim=True)
    u = d * torch.rsqrt((d ** 2).mean((1, 2, 3), keepdim=True) + 1e-5) * p[0] + p[1]
    ref = torch.autograd.grad(torch.relu(u), [z64] + p, dy.double())
    # one rounding of each stored bf16 value; fp32: coefficients with a few roundings, at most 16 of 2^-24, and short chains
    assert rel(dz, ref[0]) <= (2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -20)
    if dga is not None:
        assert rel(dga, ref[1] + 1.0) <= 2.0 ** -20
    if dbe is not None:
        assert rel(dbe, ref[2] + 2.0) <= 2.0 ** -20


@pytest.mark.parametrize("wanted", ["both", "gamma", "none"])
@pytest.mark.parametrize("shape", [(1, 5, 6, 7, 32), (3, 4, 5, 6, 64), (19, 4, 4, 4, 128)], ids=str)
def test_gate_bwd_samples(L, shape, wanted):
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    n, c, cr = shape[0], shape[4], 8

    def rnd(*s):
        return torch.randn(s, generator=g, device="cuda")

    z, dy = rnd(*shape), rnd(*shape)
    z64 = z.double()
    st = torch.stack([z64.mean((1, 2, 3)), torch.rsqrt(z64.var((1, 2, 3), unbiased=False) + 1e-5)], -1).float().contiguous()
    w1, b1, w2, b2, ga, be = rnd(cr, c) * c ** -0.5, rnd(cr) * 0.1, rnd(c, cr) * cr ** -0.5, rnd(c) * 0.1, rnd(c) * 0.1 + 1, rnd(c) * 0.1
    y, dz, gate = torch.empty_like(z), torch.empty_like(z), torch.empty((n, 4 * c + cr), device="cuda")
    dga = torch.ones((c,), device="cuda") if wanted != "none" else None
    dbe = torch.full((c,), 2.0, device="cuda") if wanted == "both" else None
    L.lamp_inorm_relu_se(z, st, w1, w2, y, gate, b1=b1, b2=b2, gamma=ga, beta=be)
    L.lamp_inorm_relu_se_bwd(dy, z, st, w1, w2, gate, dz, gamma=ga, beta=be, dgamma=dga, dbeta=dbe, beta_acc=1.0)
    z64.requires_grad_(True)
    p = [ga.double().requires_grad_(True), be.double().requires_grad_(True)]
    d = z64 - z64.mean((1, 2, 3), keepdim=True)
    a = torch.relu(d * torch.rsqrt((d ** 2).mean((1, 2, 3), keepdim=True) + 1e-5) * p[0] + p[1])
    e = torch.sigmoid(torch.relu(a.mean((1, 2, 3)) @ w1.double().T + b1.double()) @ w2.double().T + b2.double())
    ref = torch.autograd.grad(a * e[:, None, None, None], [z64] + p, dy.double())
    # fp32 sums in short chains and coefficients of a few roundings; the gate's own path (two small products) adds as many again
    assert rel(dz, ref[0]) <= 2.0 ** -19
    if dga is not None:
        assert rel(dga, ref[1] + 1.0) <= 2.0 ** -19
    if dbe is not None:
        assert rel(dbe, ref[2] + 2.0) <= 2.0 ** -19
