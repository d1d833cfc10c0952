"""The matrix-core head at the edges of its class slots: one to sixteen classes, voxel counts that leave a group unfilled, with and without a
bias, labels that name no class (they add nothing but the log of the sum), against 64-bit torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def L():
    import paper_2006_12575_amd as L
    L.lib()
    return L


@pytest.mark.parametrize("classes", [1, 2, 4, 5, 7, 8, 9, 10, 11, 13, 16])
@pytest.mark.parametrize("c,dims,bias", [(32, (9, 10, 11), True), (16, (4, 8, 12), False), (64, (5, 7, 9), True)], ids=str)
def test_head_classes(L, classes, c, dims, bias):
    g = torch.Generator(device="cuda").manual_seed(classes + c)
    x = torch.relu(torch.randn((2, *dims, c), generator=g, device="cuda")).to(BF)
    wh = (torch.randn((classes, c), generator=g, device="cuda") * (2.0 / c) ** 0.5).to(BF)
    b = torch.randn((classes,), generator=g, device="cuda") if bias else None
    lab = torch.randint(-1, classes + 1, (2, *dims), generator=g, device="cuda", dtype=torch.int32)
    logits = torch.full((2, *dims, classes), 7.0, device="cuda")
    loss, dwh, db = (torch.zeros(s, device="cuda") for s in ((1,), (classes, c), (classes,)))
    dx = torch.zeros_like(x)
    L.lamp_head_ce(x, wh, b, lab, loss, logits=logits, dx=dx, dwh=dwh, dbh=db if bias else None)
    xd, wd = x.double().reshape(-1, c), wh.double()
    z = xd @ wd.t() + (b.double() if bias else 0.0)
    v, named = lab.numel(), ((lab >= 0) & (lab < classes)).reshape(-1, 1)
    hot = torch.nn.functional.one_hot(lab.clamp(0, classes - 1).reshape(-1).long(), classes).double() * named
    d = (torch.softmax(z, 1) - hot) / v
    want = (torch.logsumexp(z, 1) - (z * hot).sum(1)).mean()

    def rel(a, e):
        return ((a.double().reshape(e.shape) - e).norm() / e.norm().clamp_min(1e-30)).item()

    assert rel(logits, z) <= 1e-6 and abs(loss.item() - want.item()) <= 1e-5 * abs(want.item()) + 1e-6
    if classes > 1:   # (one class: the gradients of the labelled voxels vanish)
        # dx: dlogits rounded to bf16 (2^-9), then dx; dwh and db in fp32
        assert rel(dx, d @ wd) <= 2 * 2.0 ** -8 and rel(dwh, d.t() @ xd) <= 1e-5
        assert not bias or rel(db, d.sum(0)) <= 1e-4
