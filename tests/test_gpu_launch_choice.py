"""Which launches lbm_step picks on a lattice nobody has chosen one for: a launch of several steps where it is
faster than single steps, single steps where it is not, and the same bits either way."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, store, bc, mrt=False, u=0.0):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx + ny)
    f = [1e-3 * r.standard_normal((ny, nx)) + (u if c == 1 else 0.0) for c in range(3)]
    return Lattice(nx, ny, 0.57, f, store=store, bc=bc, mrt=(1.6, 1.4, 1.8) if mrt else None, ubase=(u, 0.0),
                   m0=(1.0, u, 0.0))


CHANNEL, BOX, PERIODIC = (1, 1, 0, 0), (1, 1, 1, 1), (0, 0, 0, 0)


@pytest.mark.parametrize("nx,ny,store,bc,kw,n,one", [
    (128, 128, "f64", BOX, {}, 2, True), (128, 128, "f16", BOX, dict(mrt=True), 2, True),
    (512, 512, "f32", PERIODIC, {}, 4, True), (1000, 1024, "f64", CHANNEL, {}, 2, True),
    (1000, 1024, "f16", CHANNEL, {}, 2, False), (1000, 1024, "f16", CHANNEL, {}, 3, True),
    (1000, 1024, "bf16", PERIODIC, dict(mrt=True), 3, False), (2048, 1024, "f16", CHANNEL, dict(mrt=True), 4, False),
    (2048, 1024, "bf16", CHANNEL, dict(u=0.05), 4, False), (3000, 80, "f16", BOX, dict(u=0.05), 2, False),
    (3000, 80, "f16", BOX, dict(u=0.05), 3, True), (2200, 2100, "f32", CHANNEL, dict(u=0.05), 2, False),
    (2200, 2100, "f32", CHANNEL, dict(u=0.05), 3, True), (3001, 2047, "f16", CHANNEL, {}, 3, False),
    (4096, 2200, "f16", PERIODIC, {}, 3, False), (4096, 2200, "f16", PERIODIC, {}, 4, True),
    (1900, 1900, "bf16", PERIODIC, dict(u=0.05), 4, True), (2560, 2560, "f16", PERIODIC, dict(u=0.05), 4, False),
    (2048, 1024, "f16", BOX, dict(mrt=True), 2, False),
    (1000, 1024, "f16", BOX, dict(mrt=True), 3, True)])
def test_one_launch_only_where_it_is_faster(nx, ny, store, bc, kw, n, one):
    """One launch leaves the buffer it read as it was; more than one write to it."""
    g, ref = _lattice(nx, ny, store, bc, **kw), _lattice(nx, ny, store, bc, **kw)
    half = g.workspace[:9 * ny * nx * {"f64": 8, "f32": 4}.get(store, 2)]
    before = half.clone()
    g.step(n)
    torch.cuda.synchronize()
    assert torch.equal(half, before) == one
    L.lbm_set_two_step(ref.ctx, -1)
    ref.step(n)
    assert torch.equal(g.populations(), ref.populations())
    g.close()
    ref.close()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
def test_mixed_runs_equal_single_steps(store):
    """Run lengths that end in a short launch, in single steps or in both, on both sides of the size rules."""
    for nx, ny, bc, kw in ((440, 440, BOX, {}), (440, 450, CHANNEL, dict(mrt=True)), (512, 512, BOX, dict(u=0.05)),
                           (640, 819, BOX, {}), (724, 725, CHANNEL, dict(u=0.05)), (1250, 1250, PERIODIC, dict(mrt=True)),
                           (100, 6000, BOX, dict(u=0.05))):
        a, b = _lattice(nx, ny, store, bc, **kw), _lattice(nx, ny, store, bc, **kw)
        L.lbm_set_two_step(b.ctx, -1)
        for n in (2, 3, 4, 5, 6, 7, 9, 10, 11):
            a.step(n)
            b.step(n)
            assert a.t == b.t
        assert torch.equal(a.populations(), b.populations()), (nx, ny)
        assert a.check_finite()
        a.close()
        b.close()
