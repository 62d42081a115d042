"""The network's activation, bf16(tanh z) for every FP32 z from 2^-30 up to where it is 1, through the forward
pass of a network that lets hidden units through exactly: each is fed z in three BF16 pieces, and the layers
after it scale by powers of two (tanh of a value scaled by 2^-40 is that value)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LO, HI = 0x30800000, 0x41400000  # 2^-30, 12


def _through(units):
    """A trainer whose output o is the activation of hidden unit units[o], whose z is the sum of inputs
    3 o .. 3 o + 2."""
    from paper_2005_08674_amd.closure import Trainer, pack_params
    p = {"W1": np.zeros((64, 96)), "b1": np.zeros(64), "W2": np.zeros((64, 64)), "b2": np.zeros(64),
         "W3": np.zeros((3, 64)), "b3": np.zeros(3)}
    for o, u in enumerate(units):
        p["W1"][u, 3 * o:3 * o + 3] = 1.0
        p["W2"][u, u] = 2.0 ** -40
        p["W3"][o, u] = 2.0 ** 40
    return Trainer(pack_params(p), max_batch=64)


@pytest.mark.parametrize("units,sign", [((0, 1, 2), 1.0), ((3, 22, 61), -1.0)])
def test_activation_is_tanh_rounded_to_bf16(units, sign):
    """Equal to the FP64 tanh rounded to BF16, or to the other neighbour where that lies within 2 FP32 ulps of
    the middle (the FP32 tanh that decides there is itself not exact)."""
    tr, n = _through(units), 1 << 22
    x = torch.zeros((n, 96), dtype=torch.bfloat16, device="cuda")
    close = 0
    for first in range(LO, HI, 3 * n):
        bits = torch.arange(first, first + 3 * n, device="cuda", dtype=torch.int64).to(torch.int32)
        z = sign * bits.view(torch.float32)
        rest = z.clone()
        for k in range(3):
            piece = rest.to(torch.bfloat16)
            x[:, k:9:3] = piece.view(n, 3)
            rest -= piece.float()
        assert not rest.any()
        got = tr.forward(x).view(-1)
        exact = torch.tanh(z.double())
        want = exact.float().to(torch.bfloat16).float()
        bad = (got != want).nonzero().view(-1)
        ulp = torch.ldexp(torch.ones_like(exact[bad]), torch.frexp(exact[bad])[1] - 24)
        middle = 0.5 * (got[bad].double() + want[bad].double())
        assert ((exact[bad] - middle).abs() <= 2 * ulp).all(), (hex(first), bad[:5])
        # and that neighbour is the next BF16 value
        assert ((got[bad].view(torch.int32) - want[bad].view(torch.int32)).abs() == 1 << 16).all()
        close += bad.numel()
    print(f"{close} of {HI - LO} round the other way", flush=True)
    assert close < 1e-4 * (HI - LO)
    tr.close()
