"""Large batches on grids whose rows divide 256 evolve two modes of one column and plane per lane, sharing q_x and
the step's coefficients.  The same pulses in a batch with a grid that does not allow it run one mode per
lane.  Both do the same arithmetic: f and J must agree bit for bit; the per-mode bar of the oracle holds."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import assert_modes, host  # noqa: E402


@pytest.mark.parametrize("dt", [0.05, 0.3, 0.9])
@pytest.mark.parametrize("n,pz", [((1, 512, 256), (-0.4, 0.9)), ((2, 256, 256), (-0.4, 0.9)), ((64, 64, 64), (-0.8, 0.8)),
                                  ((128, 4, 256), (0.0, 1.0)), ((256, 2, 256), (-0.4, 0.9))], ids=str)
def test_pairs_match_single_modes_bitwise(orc, n, pz, dt):
    nt = 150
    grid = W.grid(n, (-1.3, -0.9, pz[0]), (1.1, 1.4, pz[1]))
    spec = W.pulse_spec(n_s=4, T=dt * nt, nt=nt, norm_value=0.2)
    c = W.draw_coeff(n[0], 3, 4)
    M = W.n_modes(grid)
    J, f = api.evaluate([spec] * 2, [grid] * 2, c[:2], want_f=True)
    Jm, fm = api.evaluate([spec] * 3, [grid, grid, W.grid((3, 5, 1), (-1, -1, 0.0), (1, 1, 0.0))], c, want_f=True)
    assert torch.equal(J, Jm[:2]) and torch.equal(f, fm[:2 * M])
    A, edge, _, _ = api.synth([spec], c[:1])
    p, _ = orc.grid_points(grid)
    sel = W.sample_mode_indices(n[0], M, 64)
    assert_modes(host(f)[sel], orc.evolve_points(host(A), host(edge)[0], dt, p[sel]), nt, f"{n} dt {dt}")
