"""A captured call on pulses that differ replays with the descriptors it was captured with, whatever the host's
memory holds by then."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import dev  # noqa: E402


@pytest.mark.parametrize("pulses", [8, 9, 17, 64])
def test_replay_of_uneven_batch(pulses):
    specs = [W.pulse_spec(n_s=4, T=0.1 * (100 + 7 * i), nt=100 + 7 * i, norm_value=0.2) for i in range(pulses)]
    grids = [W.grid((3 + i % 5, 4, 2), (-1.0, -0.8, -0.4), (1.0, 1.1, 0.9)) for i in range(pulses)]
    c = dev(W.draw_coeff(pulses, pulses, 4).ravel())
    J0, f0 = api.evaluate(specs, grids, c, want_f=True)
    A = torch.empty((api.table_rows(specs), 2), dtype=torch.float64, device="cuda")
    e = torch.empty((pulses, 2, 2), dtype=torch.float64, device="cuda")
    J, f = torch.empty_like(J0), torch.empty_like(f0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.po_evaluate(specs, grids, c, A, e, J, f=f)
    for _ in range(3):
        api.evaluate(specs[::-1], grids[::-1], c)  # eager work of other pulses between the replays
        J.zero_()
        f.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(J, J0) and torch.equal(f, f0)
