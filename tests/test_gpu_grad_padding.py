"""Yield gradient on grids whose last 256-mode item is not full, with momenta so spread that a step polynomial
chosen for the last block's modes is far outside its range at the grid's first mode: lanes without a mode
must not reach J, the table gradient or the edge terms."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_gradient import assert_grad  # noqa: E402
from test_gpu_parity import dev, host  # noqa: E402


@pytest.mark.parametrize("dt,n,lo,hi", [(0.3, (1, 1, 700), (0.0, 0.0, -15.0), (0.0, 0.0, 0.0)),
                                        (0.25, (1, 1, 700), (0.0, 0.0, -20.0), (0.0, 0.0, 0.0)),
                                        (0.3, (1, 1, 1399), (0.0, 0.0, -15.0), (0.0, 0.0, 15.0)),
                                        (0.3, (17, 13, 9), (-1.0, -1.0, -8.0), (1.0, 1.0, 8.0)),
                                        (0.3, (1, 700, 1), (0.2, -15.0, 0.0), (0.2, 0.0, 0.0))], ids=str)
def test_lanes_without_a_mode_do_not_reach_the_gradient(orc, dt, n, lo, hi):
    nt = 200
    spec, grid = W.pulse_spec(n_s=4, T=dt * nt, nt=nt, norm_value=0.1), W.grid(n, lo, hi)
    A, edge, _, _ = api.synth([spec], W.draw_coeff(3, 1, 4))
    gA, ge = torch.empty_like(A), torch.empty_like(edge)
    J = torch.empty(1, dtype=torch.float64, device="cuda")
    api.po_yield_gradient([spec], [grid], A, edge, gA, J=J, gedge=ge)
    f, J2 = api.evolve([spec], [grid], A, edge)
    J, J2, f = host(J), host(J2), host(f)
    # the same states, projected in another form: each amplitude sqrt(f) within a few units of 2^-53
    assert abs(J[0] - J2[0]) <= 1e-12 * J2[0] + 1e-14 * J2[0] / f.sum() * np.sqrt(f).sum(), (J, J2)
    ent = np.concatenate([[0, 1, 2 * nt - 1], W.sample_mode_indices(1, 2 * nt, 8), 2 * nt + np.arange(4)])
    got = np.concatenate([host(gA).ravel(), host(ge).ravel()])[ent]
    assert_grad(got, orc.grad_table_fd(host(A), host(edge)[0], dt, grid, ent), f"dt {dt} {n}")
