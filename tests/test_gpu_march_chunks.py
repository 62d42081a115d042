"""The marches at sizes where the number of their chunks follows the GPU's blocks (more chunks than the shape's
rows give, as many, or fewer) and the last run of items is short, against single-step launches: every stored
population the same bits."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, store, mrt):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx + ny)
    f = [1e-3 * r.standard_normal((ny, nx)) for _ in range(3)]
    return Lattice(nx, ny, 0.57, f, store=store, mrt=(1.6, 1.4, 1.8) if mrt else None)


# chunks of the 12-row shapes of 64, 96 and 128 rows, by the shape and as taken: 11, 8, 6 -> 37; 23, 15, 12 -> 39, 17,
# 17; 16, 11, 8 -> 16, 12, 8; 16, 11, 8 -> 27; 11, 8, 6 -> 18, 7, 7; as 1000 x 999 FP32; 2, 2, 1 -> 5; 16, 11, 8 -> 54
@pytest.mark.parametrize("nx,ny,store", [(700, 701, "f32"), (1448, 1448, "f32"), (2048, 1024, "f32"), (1000, 999, "f32"),
                                         (1501, 701, "f64"), (1000, 999, "f16"), (128, 130, "bf16"), (97, 1003, "f64")])
def test_march_chunks_equal_single_steps(nx, ny, store):
    for mrt in (False, True):
        ref = _lattice(nx, ny, store, mrt)
        L.lbm_set_two_step(ref.ctx, -1)
        L.lbm_enable_timing(ref.ctx, True)
        ref.step(6)
        assert L.lbm_kernel_times(ref.ctx)[1] == 6  # single-step launches
        want = ref.populations()
        ref.close()
        for shape in range(L.lbm_two_step_count()):
            name = L.lbm_two_step_describe(shape)
            if not name.startswith("3step") or "+march" not in name:
                continue
            g = _lattice(nx, ny, store, mrt)
            L.lbm_set_two_step(g.ctx, shape)
            g.step(6)
            assert torch.equal(g.populations(), want), (name, mrt)
            g.close()


@pytest.mark.parametrize("nx,ny,store", [(700, 701, "f32"), (417, 300, "bf16"), (330, 500, "f64")])
def test_march_with_closure_equals_single_steps(nx, ny, store):
    """The border of the inner part, cut into shorter pieces than the middle's chunks, with every node past the
    gate and with few of them."""
    from paper_2005_08674_amd.closure import Trainer
    tr = Trainer(max_batch=64, seed=5)
    tr.set_normalization(np.zeros(96, np.float32), np.full(96, 0.5, np.float32), np.full(3, 0.02, np.float32))
    for kmin in (0.0, 4.0):
        blob = tr.export(50.0, 1.0, kmin)
        want = None
        for shape in [-1] + [i for i in range(L.lbm_two_step_count()) if "3step" in L.lbm_two_step_describe(i)]:
            g = _lattice(nx, ny, store, False)
            L.lbm_set_closure(g.ctx, blob.data_ptr(), 1)
            try:
                L.lbm_set_two_step(g.ctx, shape)
            except L.LbmError:
                assert store == "f64"  # the level arrays of the taller tiles
                g.close()
                continue
            g.step(9)
            got = g.populations()
            want = got if want is None else want
            assert torch.equal(got, want), (kmin, shape)
            g.close()
