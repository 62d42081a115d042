"""The launches lbm_step chooses by itself (several steps per launch until a shape is chosen) against
single-step launches: every stored population the same bits, at the smallest lattices, at tile
remainders, on both sides of each size rule, for every edge type, storage format, collision model and
NSBC reading."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu

EDGES = [(1, 1, 1, 1), (1, 1, 0, 0), (0, 0, 1, 1), (0, 0, 0, 0), (2, 1, 0, 0), (2, 2, 0, 0)]


def _pair(nx, ny, store, bc, mrt, other):
    """(lattice left to the library, the same on single-step launches); `other`: mean flow, base velocity and
    the other NSBC readings."""
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx * 7 + ny)
    u = (0.08, 0.02) if other else (0.0, 0.0)
    f = [1e-3 * r.standard_normal((ny, nx)), u[0] + 1e-3 * r.standard_normal((ny, nx)),
         u[1] + 1e-3 * r.standard_normal((ny, nx))]
    kw = dict(store=store, bc=bc, mrt=(1.6, 1.4, 1.8) if mrt else None, ubase=u, m0=(1.0, *u),
              uw=(u[0] + 1e-3, u[1]) if 2 in bc else None)
    if other:
        kw.update(grad_order=2, corner_mode=1, corr_mode=1, beta=0.2)
    a, b = (Lattice(nx, ny, 0.57, f, **kw) for _ in range(2))
    L.lbm_set_two_step(b.ctx, -1)
    return a, b


def _check(a, b, runs):
    for n in runs:
        a.step(n)
        b.step(n)
        assert a.t == b.t
        assert torch.equal(a.populations(), b.populations()), n
    assert a.check_finite()
    a.close()
    b.close()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("bc", EDGES)
def test_chosen_launches_equal_single_steps(store, bc):
    # 17: below the smallest tile's reach; 18: the smallest; then remainders of every tile, and sizes on
    # both sides of 256 (FP64) or 512 tiles of 8 x 8 and of 256 or 1024 of 16 x 16
    for nx, ny in ((17, 19), (18, 18), (26, 27), (41, 30), (61, 133), (128, 128), (129, 128), (181, 185), (250, 257),
                   (300, 241), (520, 515)):
        for mrt, other in ((False, False), (True, False), (False, True)):
            a, b = _pair(nx, ny, store, bc, mrt, other)
            _check(a, b, (2, 5, 1, 9))


@pytest.mark.parametrize("store,nx,ny", [("f16", 723, 725), ("bf16", 733, 719), ("f16", 2050, 1030),
                                         ("f32", 2047, 1024), ("f32", 2050, 1030), ("f64", 2050, 1030)])
def test_large_lattices_equal_single_steps(store, nx, ny):
    a, b = _pair(nx, ny, store, (1, 1, 1, 1), False, True)
    _check(a, b, (2, 7))


def test_an_explicit_choice_is_kept():
    """Timing counts one launch per single step, and an explicit -1 stays with them."""
    a, b = _pair(64, 64, "f32", (1, 1, 1, 1), False, False)
    assert L.lbm_get_two_step(a.ctx) == -1
    for lat in (a, b):
        L.lbm_enable_timing(lat.ctx, True)
        lat.step(6)
        assert L.lbm_kernel_times(lat.ctx)[1] == 6
        L.lbm_enable_timing(lat.ctx, False)
    _check(a, b, (6,))
