"""A process's first call may come while a stream capture is under way: the library's scratch pool is then
created without ending the capture."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import torch
from paper_1704_08919_amd import api, workloads as W
w = W.single_pulse(0)
s, g = [dict(w["specs"][0], nt=1000)], w["grids"]
c = torch.as_tensor(w["coeff"].ravel(), dtype=torch.float64, device="cuda")
A, e, J = (torch.zeros(n, dtype=torch.float64, device="cuda") for n in ((1000, 2), (1, 2, 2), 1))
A2, e2 = torch.empty_like(A), torch.empty_like(e)
other = torch.cuda.Stream()
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    if {captured}:
        api.po_evaluate(s, g, c, A, e, J)
    else:
        J.fill_(7.0)
        api.po_pulse_synth(s, c, A2, e2, stream=other)
torch.cuda.synchronize()
eager = torch.zeros_like(J)
api.po_evaluate(s, g, c, A, e, eager)
for _ in range(3):
    junk = torch.randn(1 << 20, device="cuda").sum().item()
    J.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert J.item() == (eager.item() if {captured} else 7.0)
print("child done")
"""


@pytest.mark.parametrize("captured", [True, False], ids=["captured call", "call beside a capture"])
def test_first_call_under_capture(captured):
    r = subprocess.run([sys.executable, "-c", CHILD.format(captured=captured)], cwd=ROOT, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "child done" in r.stdout, r.stderr[-2000:]
