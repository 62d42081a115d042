"""Edge tiles of the marched three-step sweeps (64-wide tiles along the bottom and top, narrow ones along
the sides, overlapping last tiles and strips) against single steps: every stored population the same bits
around the smallest lattices that march, where the last tile or strip moves back, and with both readings of NSBC."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu

# 95 x 71 falls back to whole tiles for both tile heights, 96 x 48 marches with 8 rows only, 96 x 72 with both;
# then one strip more, side tiles that end a row before, at and after the last, and three chunks
SIZES = [(95, 71), (96, 47), (96, 48), (96, 72), (97, 73), (159, 119), (160, 120), (161, 121), (224, 201), (225, 420)]


def _lattice(nx, ny, store, **kw):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx * 7 + ny)
    u = (0.05, -0.02)
    f = [1e-3 * r.standard_normal((ny, nx)), u[0] + 1e-3 * r.standard_normal((ny, nx)),
         u[1] + 1e-3 * r.standard_normal((ny, nx))]
    return Lattice(nx, ny, 0.57, f, store=store, ubase=u, m0=(1.0, *u), beta=0.2, **kw)


def _march_shapes():
    names = [L.lbm_two_step_describe(i) for i in range(L.lbm_two_step_count())]
    return [(i, n) for i, n in enumerate(names) if n.startswith("3step") and "+march" in n]


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("kw", [dict(), dict(mrt=(1.6, 1.4, 1.8), grad_order=2, corner_mode=1, corr_mode=1)])
def test_march_edges_equal_single_steps(store, kw):
    for nx, ny in SIZES:
        ref = _lattice(nx, ny, store, **kw)
        L.lbm_set_two_step(ref.ctx, -1)
        ref.step(9)
        want = ref.populations()
        for shape, name in _march_shapes():
            g = _lattice(nx, ny, store, **kw)
            try:
                L.lbm_set_two_step(g.ctx, shape)
            except L.LbmError:
                assert store == "f64"  # the level arrays of the taller tiles
                continue
            g.step(9)
            assert torch.equal(g.populations(), want), (nx, ny, name)
            g.close()
        ref.close()


@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
def test_march_edges_with_closure_equal_single_steps(store):
    from paper_2005_08674_amd.closure import Trainer
    tr = Trainer(max_batch=64, seed=5)
    tr.set_normalization(np.zeros(96, np.float32), np.full(96, 0.5, np.float32), np.full(3, 0.02, np.float32))
    blob = tr.export(50.0, 1.0, 0.0)
    for nx, ny in SIZES:
        ref = _lattice(nx, ny, store)
        L.lbm_set_closure(ref.ctx, blob.data_ptr(), 1)
        L.lbm_set_two_step(ref.ctx, -1)
        ref.step(12)
        want = ref.populations()
        for shape, name in _march_shapes():
            g = _lattice(nx, ny, store)
            L.lbm_set_closure(g.ctx, blob.data_ptr(), 1)
            try:
                L.lbm_set_two_step(g.ctx, shape)
            except L.LbmError:
                assert store == "f64"
                continue
            g.step(12)
            assert torch.equal(g.populations(), want), (nx, ny, name)
            g.close()
        ref.close()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
def test_ensemble_of_marched_and_tiled_members_equals_single_steps(store):
    """Members on both sides of the size from which an ensemble's three-step sweep marches, BGK and MRT."""
    from paper_2005_08674_amd.ensemble import Ensemble, member_params
    members, fields = [], []
    for k, (nx, ny) in enumerate(SIZES + [(64, 20), (300, 64)]):
        members.append(member_params(nx, ny, 0.57, store=store, mrt=(1.6, 1.4, 1.8) if k % 3 == 2 else None))
        r = np.random.default_rng(nx * 7 + ny)
        fields.append(tuple(1e-3 * r.standard_normal((ny, nx)) for _ in range(3)))
    ref = Ensemble(members, fields)
    ref.step(12)
    want = [ref.populations(m) for m in range(len(members))]
    ref.close()
    for shape in range(L.lbm_two_step_count()):
        name = L.lbm_two_step_describe(shape)
        if not (name.startswith("3step:64x12") or name.startswith("3step:64x8")) or "+march" in name:
            continue
        e = Ensemble(members, fields)
        e.set_two_step(shape)
        e.step(6)
        e.step_graph(6)
        for m in range(len(members)):
            assert np.array_equal(e.populations(m), want[m]), (members[m].nx, members[m].ny, name)
        e.close()
