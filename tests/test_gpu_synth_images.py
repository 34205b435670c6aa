"""Pulse synthesis gives a time point together with its images t -> -t and, for an even number of steps, t -> t + T/2.
Table lengths where the images meet, end a workgroup of 256 base points or a chunk of 256 steps; bands
that begin at harmonic 0, an odd and an even one; all normalisations.  Tables and scale against the oracle at the
synthesis bars (1e-12 of the maximum, 1e-13); the chunk ranges that come with the tables against those of
the finished table, through the evolution's choice of series: f must agree bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import host  # noqa: E402

NORMS = {"peak": (W.NORM_PEAK, 0.4), "energy": (W.NORM_ENERGY, 2.5), "none": (W.NORM_NONE, 0.0)}


@pytest.mark.parametrize("norm", list(NORMS))
@pytest.mark.parametrize("nt", [2, 3, 4, 6, 7, 14, 255, 256, 258, 511, 514, 1000, 1023, 1024, 1026, 2050])
def test_images_match_oracle(orc, nt, norm):
    kind, value = NORMS[norm]
    T = 0.4 * nt
    dw = 2 * np.pi / T
    for first in (0, 1, 2):
        lines = max(1, min(40, nt // 4))
        spec = W.pulse_spec(n_s=5, order=3, omega_min=first * dw, omega_max=(first + lines) * dw, T=T, nt=nt, norm=kind,
                            norm_value=value)
        c = W.draw_coeff(nt + first, 1, 5)
        A, edge, scale, E = api.synth([spec], c, want_E=True)
        Ar, Er, er, sr = orc.synth(spec, c[0])
        what = f"nt {nt} first {first}"
        assert abs(host(scale)[0] - sr) <= 1e-13 * abs(sr), what
        assert np.max(np.abs(host(A) - Ar)) <= 1e-12 * np.max(np.abs(Ar)), what
        assert np.max(np.abs(host(E) - Er)) <= 1e-12 * np.max(np.abs(Er)), what
        grid = W.sheet_grid(12, 9, 2.5)
        J, f = api.evaluate([spec], [grid], c, want_f=True)
        f2, J2 = api.evolve([spec], [grid], A, edge)
        assert torch.equal(f, f2) and torch.equal(J, J2), what
