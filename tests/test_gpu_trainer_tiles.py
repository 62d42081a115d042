"""The trainer's kernels at the sizes where their tiling can go wrong: part-filled tiles of 64 samples,
more tiles than blocks, row lists with entries outside the samples, and sample counts and addresses that
leave remainders in the statistics, the packing and the forward pass."""
import numpy as np
import pytest
import torch

from oracle import mlp as M

pytestmark = pytest.mark.gpu


def _params(seed):
    rng = np.random.default_rng(seed)
    p = M.init_params(seed)
    for k, n in (("b1", 64), ("b2", 64), ("b3", 3)):
        p[k] = 0.1 * rng.standard_normal(n)
    return {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}


@pytest.mark.parametrize("batch", [1, 15, 17, 63, 64, 65, 16384, 16385, 40000])
def test_gradients_at_tile_edges(batch):
    """Every gradient entry within 1e-3 of its tensor's largest (the bar of the 1000-sample test: FP32
    accumulation and activations that round to the other BF16 value stay well below it), the loss within
    1e-4.  Every seventh row of the list lies outside the samples and must count as an empty sample."""
    from paper_2005_08674_amd.closure import Trainer, pack_params, unpack_params
    rng = np.random.default_rng(batch)
    n = 3000
    X = M.bf16_round(rng.standard_normal((n, 96)))
    T = rng.standard_normal((n, 3)).astype(np.float32).astype(np.float64)
    rows = rng.integers(0, n, batch).astype(np.int32)
    if batch > 7:
        rows[3::14] = -1
        rows[10::14] = n
    ok = (rows >= 0) & (rows < n)
    p = _params(batch)
    tr = Trainer(pack_params(p), max_batch=-(-batch // 64) * 64)
    g, loss = tr.grads(torch.tensor(X, dtype=torch.bfloat16, device="cuda"),
                       torch.tensor(T, dtype=torch.float32, device="cuda"), rows=torch.from_numpy(rows).cuda())
    # an empty sample for the oracle: zero inputs whose target is the network's own output (zero error), so
    # that the batch size, and with it the rounding of every output gradient to BF16, is the same
    y0, _ = M.forward(p, np.zeros((1, 96)), bf16=True)
    xs = np.where(ok[:, None], X[np.where(ok, rows, 0)], 0.0)
    ts = np.where(ok[:, None], T[np.where(ok, rows, 0)], y0)
    lo, go = M.loss_and_grads(p, xs, ts, bf16=True)
    assert loss == pytest.approx(lo, rel=1e-4)
    gu = unpack_params(g)
    worst = {k: float(np.abs(gu[k] - go[k]).max() / np.abs(go[k]).max()) for k in go}
    assert max(worst.values()) < 1e-3, worst


@pytest.mark.parametrize("n,shift", [(2, 0), (31, 1), (33, 3), (257, 2), (8193, 1), (70001, 0)])
def test_statistics_packing_and_forward_at_ragged_sizes(n, shift):
    """Mean and 1/std within two FP32 ulps of numpy's fp64 (the sums are fp64), packed inputs the same
    bits as torch's FP32 expression, and the forward pass of a sample the same bits wherever it sits;
    `shift` moves the inputs' address off 16 bytes."""
    from paper_2005_08674_amd.closure import Trainer
    rng = np.random.default_rng(n)
    raw = rng.standard_normal((n, 96)).astype(np.float32) + 0.5
    raw[:, 87:] = 0.0
    res = rng.standard_normal((n, 3)).astype(np.float32)
    hold = torch.zeros(n * 96 + shift, device="cuda")
    feat = hold[shift:].view(n, 96)
    feat.copy_(torch.from_numpy(raw))
    resid = torch.from_numpy(res).cuda()
    tr = Trainer(seed=1, max_batch=64)
    tr.fit_normalization(feat, resid)
    mean, inv, scale = tr.normalization()
    f = raw[:, :87].astype(np.float64)
    tol = 2 * 2.0 ** -23
    assert np.allclose(mean[:87], f.mean(0), rtol=tol, atol=tol * np.abs(f).max())
    assert np.allclose(inv[:87], 1.0 / f.std(0), rtol=tol)
    assert np.allclose(scale, np.sqrt((res.astype(np.float64) ** 2).mean(0)), rtol=tol)
    x, t = tr.pack(feat, resid)
    m, i, s = (torch.from_numpy(v).cuda() for v in (mean, inv, scale))
    assert torch.equal(x, ((feat - m) * i).to(torch.bfloat16))
    assert torch.equal(t, resid / s)
    y = tr.forward(x)
    pick = torch.from_numpy(rng.permutation(n)[:100]).cuda()
    assert torch.equal(tr.forward(x[pick].contiguous()), y[pick])
