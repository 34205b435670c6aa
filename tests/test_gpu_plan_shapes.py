"""Plans of batches too large for the time-split form (more than 448 items of 256 modes): every launch shape runs
its own kernel there, and gives the default launch's bits.  Small batches are not tuned, and what is
cached for a batch does not serve one whose modes are counted otherwise."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08919_amd import api  # noqa: E402
from paper_1704_08919_amd import workloads as W  # noqa: E402

from test_gpu_parity import dev, host  # noqa: E402
from test_gpu_plan import CONFIGS, small_uneven_batch  # noqa: E402

FILL = [W.sheet_grid(250, 460, 1.0), W.grid((60, 50, 77), (-1, -1, -0.8), (1, 1, 0.8))]  # 450 and 458 items


def large_uneven_batch(seed, fill):
    specs, grids, _ = small_uneven_batch(seed)
    specs, grids = specs + [W.pulse_spec(n_s=8, T=30.0, nt=300, norm_value=0.1)], grids + [fill]
    return specs, grids, W.draw_coeff(seed, len(specs), 8)


@pytest.mark.parametrize("cfg", CONFIGS + [dict(threads=128, modes_per_lane=1, persistent=1)], ids=str)
@pytest.mark.parametrize("fill", FILL, ids=["sheet", "mirrored"])
def test_every_shape_matches_the_default_launch_bitwise(cfg, fill):
    specs, grids, coeff = large_uneven_batch(1, fill)
    J0, f0 = api.evaluate(specs, grids, coeff, want_f=True)
    dc, J, f = dev(coeff.ravel()), torch.empty_like(J0), torch.empty_like(f0)
    plan = api.Plan(specs, grids, config=cfg)
    for k in range(3):  # the queue's counter starts anew on every replay
        J.zero_()
        f.zero_()
        plan.evaluate(dc, J, f)
        junk = torch.randn(1 << 20, device="cuda").sum()  # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(J, J0) and torch.equal(f, f0), k
        del junk
    A, edge, _, _ = api.synth(specs, coeff)
    f1, J1 = torch.zeros_like(f0), torch.zeros_like(J0)
    api.po_evolve_modes(specs, grids, A, edge, f=f1, J=J1, plan=plan)
    assert torch.equal(J1, J0) and torch.equal(f1, f0)
    plan.close()
    assert np.all(np.isfinite(host(f0)))


def test_large_batch_is_tuned_and_cached(tmp_path):
    specs, grids, coeff = large_uneven_batch(2, FILL[0])
    cache = str(tmp_path / "tune.txt")
    cfgs = []
    for _ in range(2):
        plan = api.Plan(specs, grids, cache_path=cache)
        cfgs.append(plan.config)
        J = torch.empty(len(specs), dtype=torch.float64, device="cuda")
        plan.evaluate(dev(coeff.ravel()), J)
        plan.close()
        assert torch.equal(J, api.evaluate(specs, grids, coeff)[0])
    assert cfgs[0] == cfgs[1] and len(open(cache).read().splitlines()) == 1


def test_cache_tells_symmetric_batches_from_others(tmp_path):
    """480 items where p_z is not symmetric, 240 (the time-split form, not tuned) where it is."""
    cache = str(tmp_path / "tune.txt")
    spec = [W.pulse_spec(n_s=4, T=30.0, nt=300, norm_value=0.1)]
    for lines, lo in ((1, -0.8), (2, -0.3)):
        plan = api.Plan(spec, [W.grid((64, 64, 30), (-1, -1, lo), (1, 1, 0.8))], cache_path=cache)
        if lines == 1:
            cfg = plan.config
            assert (cfg["threads"], cfg["modes_per_lane"], cfg["persistent"]) == (256, 1, 0)
        plan.close()
        keys = [x.split()[0] for x in open(cache).read().splitlines()]
        assert len(keys) == lines and len(set(keys)) == lines


def test_small_batch_keeps_the_request():
    specs, grids, _ = small_uneven_batch(3)
    plan = api.Plan(specs, grids, config=dict(persistent=1))
    assert plan.config["persistent"] == 1
    plan.close()
