"""Every launch path against single-step launches proper: the reference lattice is put on single steps and the
timing counters assert that it ran them (a lattice left alone takes several steps per launch)."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import autotune
from paper_2005_08674_amd import lbm as L
from paper_2005_08674_amd import workloads as W

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, store, bc=(1, 1, 1, 1), mrt=None, **kw):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx * 3 + ny)
    f = [1e-3 * r.standard_normal((ny, nx)) + u for u in (0.0, 0.03, -0.02)]
    return Lattice(nx, ny, 0.57, f, store=store, bc=bc, mrt=mrt, beta=0.2, m0=(1.0002, 0.03, -0.02),
                   ubase=(0.03, -0.02), uw=(0.031, -0.02) if 2 in bc else None, **kw)


def _single_steps(lat, n):
    """n steps as n launches; the populations."""
    L.lbm_set_two_step(lat.ctx, -1)
    L.lbm_enable_timing(lat.ctx, True)
    lat.step(n)
    assert L.lbm_kernel_times(lat.ctx)[1] == n and L.lbm_two_step_times(lat.ctx)[1] == 0
    L.lbm_enable_timing(lat.ctx, False)
    return lat.populations()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (61, 5), (203, 77), (241, 129), (480, 257), (1000, 999)])
def test_every_multi_step_shape(nx, ny, store):
    """11 steps: launches of three with a remainder of two, or of two with a remainder of one."""
    for mrt in (None, (1.6, 1.4, 1.8)):
        ref = _lattice(nx, ny, store, mrt=mrt)
        want = _single_steps(ref, 11)
        ref.close()
        for shape in range(L.lbm_two_step_count()):
            g = _lattice(nx, ny, store, mrt=mrt)
            try:
                L.lbm_set_two_step(g.ctx, shape)
            except L.LbmError:
                name = L.lbm_two_step_describe(shape)
                assert name.startswith("3step") and (nx < 64 or ny < 20 or store == "f64"), name
                g.close()
                continue
            g.step(11)
            assert torch.equal(g.populations(), want), (L.lbm_two_step_describe(shape), mrt)
            g.close()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("bc", [(1, 1, 1, 1), (2, 1, 0, 0), (0, 0, 0, 0)])
def test_every_single_step_tile_and_the_separate_launches(bc, store):
    for mrt in (None, (1.6, 1.4, 1.8)):
        ref = _lattice(203, 77, store, bc, mrt)
        want = _single_steps(ref, 9)
        ref.close()
        for tile in range(L.lbm_tile_count()):
            for fused, overlap in ((True, False), (False, False), (False, True)):
                g = _lattice(203, 77, store, bc, mrt)
                L.lbm_set_tile(g.ctx, tile)
                L.lbm_set_fused(g.ctx, fused)
                L.lbm_set_overlap(g.ctx, overlap)
                g.step(9)
                assert torch.equal(g.populations(), want), (L.lbm_tile_describe(tile), fused, overlap, mrt)
                g.close()


@pytest.mark.parametrize("store", ["f32", "f16"])
def test_full_size_4096_tuned_and_own_launches(store):
    """4096^2 in the cached launch and in the library's own, 32 steps (a remainder of two), against 32 single steps."""
    from paper_2005_08674_amd.lattice import Lattice
    w = W.pulses_4096()
    ref = Lattice(w.nx, w.ny, w.tau, w.fields, store=store)
    want = _single_steps(ref, 32)
    ref.close()
    for tuned in (True, False):
        g = Lattice(w.nx, w.ny, w.tau, w.fields, store=store)
        if tuned and autotune.apply(g, store) is None:
            autotune.tune(g, store, reps=3, path=None)
        g.step(32)
        assert torch.equal(g.populations(), want), tuned
        g.close()
