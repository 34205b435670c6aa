"""Accuracy of f where the step angle is beyond the polynomial fits and the phases are large (large momenta or steps):
rms error against the long-double oracle.  With q = (p - A) dt it is 7.5e-16, 6.5e-14 and 1.4e-14 in the
three cases, set by the rounding of q; with q from (p - A) / e_perp, whose rounding is the same in every
step, 2.4e-15, 1.1e-13 and 3.1e-14.  The bars are 1.3 times the former."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import dev, host, say  # noqa: E402


def table(dt, nt, amp, seed):
    """Five random sines per component over the pulse: A at the step midpoints and at both ends."""
    r = np.random.default_rng(seed)
    w, ph, a = r.uniform(0.2, 3, (5, 2)) / (nt * dt) * 12, r.uniform(0, 6.28, (5, 2)), r.normal(size=(5, 2)) * amp / 3

    def A(t):
        return (a * np.sin(w * np.asarray(t)[..., None, None] + ph)).sum(-2)

    return A((np.arange(nt) + 0.5) * dt), np.stack([A(0.0), A(nt * dt)])


@pytest.mark.parametrize("dt,P,amp,nt,seed,bar", [(0.1, 30.0, 10.0, 1000, 140, 9.7e-16),
                                                  (0.02, 1000.0, 1000.0, 300, 160, 8.5e-14),
                                                  (3.0, 5.0, 3.0, 300, 180, 1.9e-14)])
def test_error_beyond_the_fits(orc, dt, P, amp, nt, seed, bar):
    spec = W.pulse_spec(n_s=4, T=dt * nt, nt=nt)
    grid = W.grid((12, 11, 8), (-P, -0.9 * P, -0.3 * P), (0.8 * P, P, 0.7 * P))
    p, _ = orc.grid_points(grid)
    sq = []
    for k in range(2):
        A, edge = table(dt, nt, amp, seed + k)
        f, _ = api.evolve([spec], [grid], dev(A), dev(edge[None]))
        sq.append(np.mean((host(f) - orc.evolve_points(A, edge, dt, p)) ** 2))
    rms = float(np.sqrt(np.mean(sq)))
    say(f"dt {dt} p to {P}: rms {rms:.2e}")
    assert rms <= bar
