"""Tables with more than 512 blocks of field statistics (nt above 262144, or 524288 where it is even), where the scale is
a kernel of its own: tables, samples and scale against the oracle at the synthesis bars (1e-12 of the
maximum, 1e-13), beside a short pulse of the same batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import host  # noqa: E402


@pytest.mark.parametrize("norm,value", [(W.NORM_PEAK, 0.3), (W.NORM_ENERGY, 2.0)], ids=["peak", "energy"])
@pytest.mark.parametrize("nt", [300001, 600002])
def test_long_table(orc, nt, norm, value):
    specs = [W.pulse_spec(n_s=4, T=20.0, nt=n, norm=norm, norm_value=value) for n in (nt, 200)]
    c = W.draw_coeff(nt, 2, 4)
    A, edge, scale, E = (host(t) for t in api.synth(specs, c, want_E=True))
    A2, _, scale2, _ = api.synth(specs, c)
    assert np.array_equal(host(A2), A) and np.array_equal(host(scale2), scale)
    Es, _, As, es, ss = (host(t) for t in api.field_samples(specs, c, (0.5,), with_end=True))
    row = 0
    for i, s in enumerate(specs):
        Ar, Er, er, sr = orc.synth(s, c[i])
        n = s["nt"]
        at, rt = slice(row, row + n), slice(row + i, row + i + n)
        for a, b, sc, ed in ((A[at], E[at], scale[i], edge[i]), (As[rt], Es[rt], ss[i], es[i])):
            assert abs(sc - sr) <= 1e-13 * sr
            assert np.max(np.abs(a - Ar)) <= 1e-12 * np.max(np.abs(Ar))
            assert np.max(np.abs(b - Er)) <= 1e-12 * np.max(np.abs(Er))
            assert np.max(np.abs(ed - er)) <= 1e-12 * np.max(np.abs(Ar))
        row += n
