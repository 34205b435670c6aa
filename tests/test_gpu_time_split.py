"""Small batches are evolved with one workgroup per (256-mode item, time segment); the segments' propagators
are then applied in order.  The same pulse inside a batch that fills the GPU is walked through segment
by segment by one workgroup.  Both do the same arithmetic: f and J must agree bit for bit, whatever the
batch, the launch shape or the entry point; and the split form meets the oracle's per-mode bar."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import assert_modes, dev, host  # noqa: E402

BIG = W.sheet_grid(250, 460, 1.0)  # 450 items: alone enough for the form without the split


@pytest.mark.parametrize("nt", [2, 63, 64, 65, 128, 700, 1000, 4096, 4100])
@pytest.mark.parametrize("n", [(1, 1, 1), (17, 13, 3), (64, 33, 4)], ids=str)
def test_split_matches_walk_bitwise(orc, nt, n):
    spec = W.pulse_spec(n_s=4, T=0.09 * nt, nt=nt, norm_value=0.2)
    other = W.pulse_spec(n_s=4, T=0.9, nt=9, norm_value=0.2)
    grid = W.grid(n, (-1.3, -0.9, -0.7), (1.1, 1.4, 0.7))
    c = W.draw_coeff(nt, 2, 4)
    J, f = api.evaluate([spec], [grid], c[:1], want_f=True)
    Jb, fb = api.evaluate([spec, other], [grid, BIG], c, want_f=True)
    M = W.n_modes(grid)
    assert torch.equal(J, Jb[:1]) and torch.equal(f, fb[:M])
    for cfg in (dict(threads=256, modes_per_lane=1, persistent=0), dict(threads=128, modes_per_lane=2, persistent=1)):
        plan = api.Plan([spec, other], [grid, BIG], config=cfg)
        Jp, fp = torch.empty_like(Jb), torch.empty_like(fb)
        plan.evaluate(dev(c.ravel()), Jp, fp)
        plan.close()
        assert torch.equal(Jp, Jb) and torch.equal(fp, fb), cfg
    A, edge, _, _ = api.synth([spec], c[:1])
    p, _ = orc.grid_points(grid)
    sel = W.sample_mode_indices(nt, M, 64)
    assert_modes(host(f)[sel], orc.evolve_points(host(A), host(edge)[0], spec["T"] / nt, p[sel]), nt, f"{nt} {n}")


def test_uneven_small_batch_matches_single_calls_bitwise():
    specs = [W.pulse_spec(n_s=4, T=0.09 * nt, nt=nt, norm_value=0.2) for nt in (300, 64, 2048)]
    grids = [W.sheet_grid(32, 32, 1.5), W.box_grid(16, 16, 4), W.grid((9, 5, 2), (-1, -1, 0.0), (1, 1, 0.9))]
    c = W.draw_coeff(4, 3, 4)
    J, f = api.evaluate(specs, grids, c, want_f=True)
    off = 0
    for i in range(3):
        Ji, fi = api.evaluate(specs[i:i + 1], grids[i:i + 1], c[i:i + 1], want_f=True)
        assert torch.equal(Ji, J[i:i + 1]) and torch.equal(fi, f[off:off + W.n_modes(grids[i])])
        off += W.n_modes(grids[i])
    assert np.all(np.isfinite(host(f)))
