"""Yield gradients whose propagators and partial sums exceed the scratch limit of 2 GiB are worked through in
groups of 256-mode items: whole pulses, or parts of one.  The sums over items go on from group to group in
the same order, so nothing depends on the groups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import host, say  # noqa: E402


def gradient(specs, grids, A, edge):
    gA, ge = torch.empty_like(A), torch.empty_like(edge)
    J = torch.empty(len(specs), dtype=torch.float64, device="cuda")
    api.po_yield_gradient(specs, grids, A, edge, gA, J=J, gedge=ge)
    return J, gA, ge


def box(nz, lo, hi):
    return W.grid((256, 256, nz), (-1.5, -1.0, lo), (1.0, 1.25, hi))


@pytest.mark.parametrize("order", [(0, 1, 2), (2, 0, 1)], ids=str)
def test_groups_of_pulses_match_single_calls_bitwise(order):
    nts = [64, 64, 200]  # 1.1 GiB, 1.1 GiB and a small one
    allg = [box(256, -0.5, 1.0), box(256, 0.25, 1.25), W.grid((17, 13, 3), (-1.3, -0.9, -0.7), (1.1, 1.4, 0.8))]
    specs = [W.pulse_spec(n_s=4, T=0.2 * nts[i], nt=nts[i], norm_value=0.3) for i in order]
    grids = [allg[i] for i in order]
    A, edge, _, _ = api.synth(specs, W.draw_coeff(5, 3, 4))
    J, gA, ge = gradient(specs, grids, A, edge)
    row = 0
    for i in range(3):
        nt = specs[i]["nt"]
        J1, gA1, ge1 = gradient(specs[i:i + 1], grids[i:i + 1], A[row:row + nt].contiguous(), edge[i:i + 1].contiguous())
        assert torch.equal(J1, J[i:i + 1]) and torch.equal(gA1, gA[row:row + nt]) and torch.equal(ge1, ge[i:i + 1]), i
        row += nt


def test_parts_of_a_pulse_add_up():
    """A box of 2^26 modes (4.6 GiB, three groups) against its quarters (one group each).  The step in p_z
    is a power of two, so the modes and their values are the same; J is a sum of positive terms over some 4000 additions in a row (5e-13), a gradient entry one of
    262144 in order (3e-11 of the terms' magnitude)."""
    nt = 64
    spec = W.pulse_spec(n_s=4, T=0.2 * nt, nt=nt, norm_value=0.3)
    A, edge, _, _ = api.synth([spec], W.draw_coeff(6, 1, 4))
    J, gA, ge = (host(t) for t in gradient([spec], [box(1024, -0.5, 1.5)], A, edge))
    parts = [[host(t) for t in gradient([spec], [box(256, lo, lo + 0.5)], A, edge)] for lo in (-0.5, 0.0, 0.5, 1.0)]
    Jq, gAq, geq = (sum(p[k] for p in parts) for k in range(3))
    say(f"J rel {abs(J[0] / Jq[0] - 1):.2e}, gA {np.abs(gA - gAq).max() / np.abs(gA).max():.2e}, "
        f"edges {np.abs(ge - geq).max() / np.abs(ge).max():.2e}")
    assert abs(J[0] - Jq[0]) <= 1e-12 * J[0]
    assert np.all(np.abs(gA - gAq) <= 1e-10 * np.abs(gA).max())
    assert np.all(np.abs(ge - geq) <= 1e-10 * np.abs(ge).max())


def test_largest_grid_fits():
    """2^30 modes at nt = 512, eight segments: 576 GB of scratch in one piece."""
    nt = 512
    spec = W.pulse_spec(n_s=4, T=0.1 * nt, nt=nt, norm_value=0.5)
    grid = W.grid((1024, 1024, 1024), (-1.0, -1.0, -0.5), (1.5, 1.25, 1.0))
    A, edge, _, _ = api.synth([spec], W.draw_coeff(7, 1, 4))
    J, gA, ge = gradient([spec], [grid], A, edge)
    _, J2 = api.evolve([spec], [grid], A, edge, want_f=False)
    J, J2 = host(J), host(J2)
    say(f"J rel {abs(J[0] / J2[0] - 1):.2e}")
    assert abs(J[0] - J2[0]) <= 1e-11 * J2[0]  # as for small grids (another form of the projection)
    assert torch.isfinite(gA).all() and torch.isfinite(ge).all()
