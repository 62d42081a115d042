"""The face rows of the 3-D launches (64 nodes per block, their loads spread over its wavefronts) at row
lengths around 64 and 128 and at the smallest sides, for every mix of NSBC and periodic faces, and the
launch shape the library picks against every shape the lattice takes."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu

MIXES = [tuple(v for a in axes for v in (a, a)) for axes in itertools.product((1, 0), repeat=3)]


def _fields(nx, ny, nz):
    r = np.random.default_rng(nx + 100 * ny)
    return [1e-3 * r.standard_normal((nz, ny, nx)) + u for u in (0.0, 0.03, -0.02, 0.01)]


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("dims", [(3, 70, 3), (63, 3, 4), (64, 4, 3), (65, 5, 4), (129, 3, 5)])
def test_face_rows_against_oracle(dims, q):
    """FP64 within the parity bar of the other 3-D tests (1e-12, velocities relative to the flow's 0.03)."""
    from paper_2005_08674_amd.lattice3d import Lattice3D
    f = _fields(*dims)
    for bc in MIXES:
        kw = dict(bc=bc, beta=0.2, m0=(1.0, 0.03, -0.02, 0.01), q=q)
        g, o = Lattice3D(*dims, 0.6, f, store="f64", **kw), oracle.Lattice3D(*dims, 0.6, *f, **kw)
        g.step(7)
        o.step(7)
        gm, om = g.moments(), o.moments()
        assert np.abs(gm[0] - om[0]).max() <= 1e-12, bc
        assert max(np.abs(gm[a] - om[a]).max() for a in (1, 2, 3)) <= 1e-12 * 0.03, bc
        g.close()


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx", [5, 64, 66, 97, 130, 256, 259])
def test_default_shape_equals_every_shape(nx, store):
    from paper_2005_08674_amd.lattice3d import Lattice3D
    for bc in ((1,) * 6, (0, 0, 1, 1, 1, 1)):
        f, ref = _fields(nx, 6, 5), None
        for shape in [None] + list(range(L.lbm3d_shape_count())):
            g = Lattice3D(nx, 6, 5, 0.6, f, store=store, bc=bc, q=19)
            try:
                if shape is not None:
                    L.lbm3d_set_shape(g.ctx, shape)
            except L.LbmError:
                g.close()
                continue
            g.step(3)
            p = g.populations()
            ref = p if ref is None else ref
            assert torch.equal(p, ref), (bc, shape)
            g.close()
