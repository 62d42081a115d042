"""lbm_step recorded into a HIP graph on a lattice nobody has chosen a launch for: a graph of an even number
of steps, replayed, goes on stepping from the state the last replay left."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,bc,steps", [(96, 64, (1, 1, 1, 1), 2), (96, 64, (1, 1, 0, 0), 4), (200, 130, (0, 0, 0, 0), 6),
                                            (2048, 1100, (1, 1, 1, 1), 2)])
def test_replays_of_an_even_number_of_steps_advance(nx, ny, bc, steps):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(5)
    f = [1e-3 * r.standard_normal((ny, nx)) for _ in range(3)]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = Lattice(nx, ny, 0.6, f, store="f32", bc=bc, stream=s)
        a.step(1)
    s.synchronize()
    b = Lattice(nx, ny, 0.6, f, store="f32", bc=bc)
    L.lbm_set_two_step(b.ctx, -1)
    b.step(1)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        a.step(steps)
    for _ in range(3):
        with torch.cuda.stream(s):
            g.replay()
        s.synchronize()
        b.step(steps)
        assert torch.equal(a.populations(), b.populations())
    # and outside a graph the lattice steps on
    a.step(5)
    s.synchronize()
    b.step(5)
    assert torch.equal(a.populations(), b.populations())
    a.close()
    b.close()
