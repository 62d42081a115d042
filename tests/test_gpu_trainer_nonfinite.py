"""Gradients where a target or an intermediate value overflows: what is non-finite stays with its output, and
the entries that do not depend on it keep the bits they have without it."""
import numpy as np
import pytest
import torch

from oracle import mlp as M

pytestmark = pytest.mark.gpu


def _grads(p, x, t):
    from paper_2005_08674_amd.closure import Trainer, pack_params, unpack_params
    tr = Trainer(pack_params(p), max_batch=128)
    g, _ = tr.grads(x, t)
    tr.close()
    return unpack_params(g)


def _samples(n):
    r = np.random.default_rng(n)
    return (torch.tensor(r.standard_normal((n, 96)), dtype=torch.bfloat16, device="cuda"),
            torch.tensor(r.standard_normal((n, 3)), dtype=torch.float32, device="cuda"))


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("n,row,out", [(64, 0, 0), (100, 99, 1), (17, 5, 2)])
def test_a_non_finite_target_stays_in_its_output(n, row, out, bad):
    x, t = _samples(n)
    p = M.init_params(3)
    good = _grads(p, x, t)
    t[row, out] = bad
    g = _grads(p, x, t)
    others = [o for o in range(3) if o != out]
    assert not np.isfinite(g["W3"][out]).any() and not np.isfinite(g["b3"][out])
    assert np.array_equal(g["W3"][others], good["W3"][others])
    assert np.array_equal(g["b3"][others], good["b3"][others])


def test_an_overflowing_hidden_gradient_stays_in_its_unit():
    """One weight of the last layer large enough that the hidden gradient of its unit, and of no other, passes
    FP32's range: the other units' rows of the second layer's gradient stay finite."""
    x, t = _samples(64)
    p = M.init_params(4)
    t[7, 0] = 3e38  # d(loss) / d(output) = 2 * 3e38 / (3 * 64) = 3e36
    p["W3"][0, 5] = 1e4
    g = _grads(p, x, t)
    rest = [k for k in range(64) if k != 5]
    assert not np.isfinite(g["W2"][5]).any() and not np.isfinite(g["b2"][5])
    assert np.isfinite(g["W2"][rest]).all() and np.isfinite(g["b2"][rest]).all()
    assert np.isfinite(g["W3"]).all()
