"""A process's first call of an entry point may come inside a graph capture: every replay gives what the eager call gives."""
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import sys
import torch
sys.path.insert(0, %r)
import paper_2006_12575_amd as L
L.lib()
torch.manual_seed(3)
kind, dt, shape, co = sys.argv[1], getattr(torch, sys.argv[2]), eval(sys.argv[3]), int(sys.argv[4])
x = torch.randn(shape, device="cuda").to(dt)
ws = torch.empty(1 << 27, dtype=torch.uint8, device="cuda")
if kind == "wgrad":
    dy, dw = torch.randn((*shape[:4], co), device="cuda").to(dt), torch.empty((co, 3, 3, 3, shape[4]), device="cuda")
    call = lambda: L.lamp_conv3d_wgrad(x, dy, dw, ws=ws)
elif kind == "fwd":
    wt, dw, st = torch.randn((co, 3, 3, 3, shape[4]), device="cuda").to(dt), torch.empty((*shape[:4], co), device="cuda", dtype=dt), torch.empty((shape[0], co, 2), device="cuda")
    call = lambda: L.lamp_conv3d_fwd(x, wt, dw, stats_out=st, ws=ws)
elif kind == "convtr all":
    wt = torch.randn((shape[4], 2, 2, 2, co), device="cuda").to(dt)
    dy, dx, db = torch.randn((shape[0], *(2 * s for s in shape[1:4]), co), device="cuda").to(dt), torch.empty_like(x), torch.empty(co, device="cuda")
    dw = torch.empty(wt.shape, device="cuda")
    call = lambda: L.lamp_convtr3d_bwd(x, wt, dy, dx=dx, dwt=dw, dbias=db, ws=ws)
else:
    wt = torch.randn((shape[4], 2, 2, 2, co), device="cuda").to(dt)
    dy, dw = torch.randn((shape[0], *(2 * s for s in shape[1:4]), co), device="cuda").to(dt), torch.empty(wt.shape, device="cuda")
    call = lambda: L.lamp_convtr3d_bwd(x, wt, dy, dwt=dw, ws=ws)
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    call()
got = []
for _ in range(3):
    dw.fill_(float("nan"))
    g.replay()
    torch.cuda.synchronize()
    got.append(dw.clone())
    (x.float() * 2).sum().item()
dw.fill_(float("nan"))
call()
torch.cuda.synchronize()
assert all(torch.equal(t, dw) for t in got) and torch.isfinite(dw).all()
print("replays equal")
"""


@pytest.mark.parametrize("kind,dtype,shape,co", [("wgrad", "bfloat16", (2, 20, 24, 32, 2), 16), ("wgrad", "bfloat16", (1, 20, 24, 28, 24), 40),
                                                 ("wgrad", "float32", (1, 20, 24, 28, 32), 32), ("convtr", "bfloat16", (1, 10, 12, 14, 16), 8),
                                                 ("fwd", "float32", (1, 10, 12, 14, 32), 32), ("convtr all", "bfloat16", (1, 10, 12, 14, 32), 16)], ids=str)
def test_first_call_in_a_capture(kind, dtype, shape, co):
    import conftest
    r = subprocess.run([sys.executable, "-c", CHILD % conftest.ROOT, kind, dtype, str(shape), str(co)], capture_output=True, text=True, timeout=90)
    assert r.returncode == 0 and "replays equal" in r.stdout, r.stderr[-2000:]
