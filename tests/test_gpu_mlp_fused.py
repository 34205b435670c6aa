"""The network kernels at the edges of their ranges against the NumPy oracle (same bf16 rounding points):
widths of one column tile, of one and two tiles per wave, the largest that one workgroup takes and the
next one (layer by layer); inputs narrower and wider than the network; one to four layers; batches that
split the weight gradients into 1, 2 and 4 parts.  Ranking and index compaction at the edges of theirs.

Tolerances: float32 against float64 sums only differ where an activation rounds to the other bf16 value,
one part in 2^8 of that activation and of what it feeds.  An activation is one of at least 32 terms, so one
flip moves an output by less than 2^-8 of the output's range (bar: 1e-2, a few flips), the loss, a mean
over the batch, by less than 1e-4, and a gradient tensor by at most 2^-8 of its norm (bar 5e-3)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from oracle import mlp as M  # noqa: E402
from paper_1704_08919_amd import api  # noqa: E402

from test_gpu_parity import dev, host, say  # noqa: E402


@pytest.mark.parametrize("n_in,width,depth,batch,max_batch", [
    (32, 32, 1, 32, 32), (96, 32, 2, 96, 128), (32, 256, 4, 64, 64), (32, 288, 2, 128, 256), (512, 512, 2, 128, 128),
    (64, 480, 3, 96, 160), (544, 64, 2, 64, 64), (32, 544, 2, 64, 96)])
def test_network_edges(n_in, width, depth, batch, max_batch):
    rng = np.random.default_rng(width + depth)
    x = rng.uniform(-1, 1, (batch, n_in))
    t = (np.sin(2 * x[:, 0]) + x[:, 1] * x[:, 2]).astype(np.float32)
    a = api.MLP(n_in, width, depth, max_batch=max_batch, seed=3)
    b = api.MLP(n_in, width, depth, max_batch=max_batch, seed=3)
    p = host(a.get_params()).astype(np.float64)
    y = host(a.forward(dev(x)))
    yr, _ = M.forward(p, x, n_in, width, depth, bf=True)
    e = np.max(np.abs(y - yr)) / np.ptp(yr)
    loss, g = a.loss_grad(dev(x), dev(t, torch.float32))
    loss, gh = float(host(loss)[0]), host(g).astype(np.float64)
    lr_, gr = M.loss_grad(p, x, t.astype(np.float64), n_in, width, depth, bf=True)
    Wg, bg = M.unpack(gh, n_in, width, depth)
    Wr, br = M.unpack(gr, n_in, width, depth)
    eg = max(np.linalg.norm(u - v) / np.linalg.norm(v) for u, v in zip([*Wg, *bg], [*Wr, *br]))
    say(f"mlp {n_in}x{width}x{depth} batch {batch}: outputs {e:.1e}, loss {abs(loss / lr_ - 1):.1e}, gradient {eg:.1e}")
    assert e <= 1e-2 and abs(loss - lr_) <= 1e-4 * lr_ and eg <= 5e-3
    # the training step is the gradient and the optimiser, bit for bit, and its weights are the next pass's
    for _ in range(2):
        la = torch.empty(1, dtype=torch.float32, device="cuda")
        b.train_step(dev(x), dev(t, torch.float32), lr=1e-3, loss=la)
        lb, g = a.loss_grad(dev(x), dev(t, torch.float32))
        a.adam_step(g, lr=1e-3)
        assert float(host(la)[0]) == float(host(lb)[0])
        assert np.array_equal(host(a.get_params()), host(b.get_params()))
        assert np.array_equal(host(a.forward(dev(x))), host(b.forward(dev(x))))
    a.close()
    b.close()


@pytest.mark.parametrize("n", [1, 31, 33, 1023, 1025, 8191, 8192])
def test_ranking_and_indices(n):
    rng = np.random.default_rng(n)
    s = rng.normal(0, 1, n).astype(np.float32)
    special = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 0.0, -1e-45, 1e-45, np.nan, np.inf], dtype=np.float32)
    s[rng.permutation(n)[:len(special)]] = special[:n]
    for k in {0, 1, n // 3, n - 1, n}:
        mask = host(api.po_topk_mask(dev(s, torch.float32), k))
        order = sorted(range(n), key=lambda i: (bool(np.isnan(s[i])), 0.0 if np.isnan(s[i]) else -s[i], i))
        ref = np.zeros(n, dtype=np.uint8)
        ref[order[:k]] = 1
        assert np.array_equal(mask, ref), k
        cnt = torch.empty(1, dtype=torch.int32, device="cuda")
        idx = host(api.po_mask_indices(dev(mask, torch.uint8), count=cnt))
        assert int(host(cnt)[0]) == k
        assert np.array_equal(idx[:k], np.flatnonzero(ref))
