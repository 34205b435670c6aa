"""The fourth-order and split-operator steps where their forms change: every series and the angle-halving path
beyond them, table lengths around the rescaling group (64 steps) and the chunk (256), and one workgroup
per (item, time segment) against one per item, which must agree bit for bit.  Reference: the long-double
oracle on the same tables, at the per-mode bar of the Dirac path (1e-9 f + 2 sqrt(f) d + d^2,
d = 4 * 2^-53 * sqrt(nt); three substeps count as three steps)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import assert_modes, dev, host  # noqa: E402

BIG = W.sheet_grid(250, 460, 1.0)  # 450 items: alone enough for one workgroup per item
POINTS = {"m4": 2, "split2": 1, "split4": 3}
CASES = {f"nt{nt}": (nt, 0.05) for nt in (2, 63, 65, 255, 257, 515)}
CASES.update({f"dt{dt:g}": (300, dt) for dt in (0.005, 0.03, 0.06, 0.1, 0.14, 0.19, 0.31, 0.41, 0.5, 0.65, 0.9)})


def run(scheme, specs, grids, A, edge):
    if scheme == "m4":
        return api.evolve_m4(specs, grids, A, edge)
    return api.evolve_split(specs, grids, int(scheme[-1]), A, edge)


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("scheme", list(POINTS))
def test_step_forms_match_oracle_and_each_other(orc, scheme, case):
    nt, dt = CASES[case]
    k = POINTS[scheme]
    r = W.rng(nt)
    t = np.arange(nt * k)[:, None] / (nt * k)
    A = sum(r.uniform(-0.2, 0.2, 2) * np.sin(2 * np.pi * m * t + r.uniform(0, 6, 2)) for m in (1, 2, 5))
    edge = r.uniform(-0.3, 0.3, (2, 2, 2))
    grid = W.grid((7, 5, 3), (-1.9, -1.4, -0.8), (1.7, 1.6, 1.1))
    specs = [W.pulse_spec(n_s=4, T=n * dt, nt=n, norm=W.NORM_NONE, norm_value=0.0) for n in (nt, 9)]
    A = A.reshape(nt, k, 2)
    f, J = run(scheme, specs[:1], [grid], dev(A), dev(edge[:1]))
    fb, Jb = run(scheme, specs, [grid, BIG], dev(np.concatenate([A, 0.1 * np.ones((9, k, 2))])), dev(edge))
    assert torch.equal(f, fb[:W.n_modes(grid)]) and torch.equal(J, Jb[:1])
    p, _ = orc.grid_points(grid)
    if scheme == "m4":
        fr = orc.evolve4_points(A, edge[0], specs[0]["T"] / nt, p)
    else:
        fr = orc.evolve_split_points(A if k > 1 else A[:, 0], edge[0], specs[0]["T"] / nt, p, order=int(scheme[-1]))
    assert_modes(host(f), fr, nt * (3 if k == 3 else 1), f"{scheme} {case}")
