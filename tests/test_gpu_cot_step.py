"""The cotangent-form evolution step (Sec. II A's exact midpoint exponential) where its forms change:
every fit variant and the angle-halving path beyond them, table lengths around the rescaling group
(64 steps) and the chunk (256), and steps small enough for the short group (dt < 2^-14) and for the
unscaled path (dt < 2^-59).  Reference: the long-double oracle on the same tables, at the per-mode
bar of the Dirac path (1e-9 f + 2 sqrt(f) d + d^2, d = 4 * 2^-53 * sqrt(nt))."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import assert_modes, dev, host  # noqa: E402

CASES = {f"nt{nt}": (nt, 0.05) for nt in (2, 3, 63, 64, 65, 129, 255, 256, 257, 515)}
CASES.update({f"dt{dt:g}": (300, dt) for dt in (0.008, 0.03, 0.06, 0.1, 0.14, 0.19, 0.31, 0.41, 0.5, 0.9)})
CASES.update({f"dt2^{k}": (300, 2.0 ** k) for k in (-14, -15, -40, -59, -60, -300)})


@pytest.mark.parametrize("case", list(CASES))
def test_step_forms_match_oracle(orc, case):
    nt, dt = CASES[case]
    r = W.rng(nt)
    t = np.arange(nt)[:, None] / nt
    A = sum(r.uniform(-0.2, 0.2, 2) * np.sin(2 * np.pi * k * t + r.uniform(0, 6, 2)) for k in (1, 2, 5))
    edge = r.uniform(-0.3, 0.3, (1, 2, 2))
    grid = W.grid((7, 5, 3), (-1.9, -1.4, -0.8), (1.7, 1.6, 1.1))
    spec = W.pulse_spec(n_s=4, T=nt * dt, nt=nt, norm=W.NORM_NONE, norm_value=0.0)
    f, _ = api.evolve([spec], [grid], dev(A), dev(edge))
    p, _ = orc.grid_points(grid)
    assert_modes(host(f), orc.evolve_points(A, edge[0], spec["T"] / nt, p), nt, case)
