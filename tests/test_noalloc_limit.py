"""The documented scratch limit of po_evaluate_noalloc (64 MiB) decides on the host, before any pointer is looked
at: which batches it refuses is part of the interface, however the library lays its scratch out."""
import ctypes

import pytest

from paper_1704_08919_amd import _lib
from paper_1704_08919_amd import workloads as W
from paper_1704_08919_amd.api import _grid_array, _spec_array


def up(x):
    return (x + 255) // 256 * 256


def documented_bytes(specs, grids):
    lines = sum(int((s["omega_max"] - s["omega_min"]) / (2 * 3.141592653589793 / s["T"]) + 1e-9) + 1 for s in specs)
    blocks = max([1] + [(s["nt"] + 256) // 256 for s in specs if s["norm"] != W.NORM_NONE])
    units = sum((W.n_modes(g) + 63) // 64 for g in grids)
    chunks = sum((s["nt"] + 255) // 256 for s in specs)
    n = len(specs)
    return up(208 * n) + up(32 * lines) + up(8 * blocks * n) + up(8 * n) + up(8 * units) + up(32 * chunks)


@pytest.mark.parametrize("norm", [W.NORM_NONE, W.NORM_PEAK, W.NORM_ENERGY])
@pytest.mark.parametrize("nt,T,n", [(131072, 100.0, (4, 4, 1)), (131071, 100.0, (4, 4, 1)), (1000, 800.0, (128, 128, 64)),
                                    (65536, 8000.0, (4, 4, 2)), (32768, 100.0, (64, 64, 64))])
def test_limit(nt, T, n, norm):
    lib = _lib.load()
    spec = W.pulse_spec(n_s=4, T=T, nt=nt, norm=norm, norm_value=0.1 if norm != W.NORM_NONE else 0.0)
    grid = W.grid(n, (-1, -1, -0.5 if n[2] > 1 else 0), (1, 1, 0.5 if n[2] > 1 else 0))
    lo, hi = 1, 4096  # largest count that the documented size lets pass
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if documented_bytes([spec] * mid, [grid] * mid) <= 64 << 20 else (lo, mid - 1)
    assert 1 < lo < 4096
    for pulses, refused in ((lo, False), (lo + 1, True)):
        st = lib.po_evaluate_noalloc(pulses, _spec_array([spec] * pulses), _grid_array([grid] * pulses), None, None, None,
                                     None, None, ctypes.c_void_p(8), None)
        assert st == _lib.PO_ERR_INVALID
        assert (b"allocation-free path holds" in lib.po_last_error()) == refused, (pulses, lib.po_last_error())
