"""Tuning a lattice whose own launches of several steps are the fastest ends on those, and the cache and the
calls that select a launch lead there and back; the bits are those of single steps throughout."""
import numpy as np
import pytest
import torch

from paper_2005_08674_amd import autotune
from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu

# sizes where those launches take less than two thirds of the next best's time
CASES = [(128, 128, "f64", (1, 1, 1, 1), None), (128, 128, "f32", (2, 1, 0, 0), (1.4, 1.4, 1.2)),
         (1501, 701, "f32", (1, 1, 0, 0), None), (600, 600, "f32", (0, 0, 0, 0), None)]


def _lattice(nx, ny, store, bc, mrt):
    from paper_2005_08674_amd.lattice import Lattice
    r = np.random.default_rng(nx)
    f = [1e-3 * r.standard_normal((ny, nx)) for _ in range(3)]
    return Lattice(nx, ny, 0.58, f, store=store, bc=bc, mrt=mrt, uw=(1e-3, 0.0) if 2 in bc else None)


def _three_steps_in_one_launch(g):
    """One launch leaves the buffer it read as it was (called in turn with an even number of launches before)."""
    half = g.workspace[:9 * g.ny * g.nx * (8 if g.params.store == L.STORE_NAMES["f64"] else 4)]
    before = half.clone()
    g.step(3)
    torch.cuda.synchronize()
    same = torch.equal(half, before)
    g.step(3)  # back to the first buffer
    return same


@pytest.mark.parametrize("nx,ny,store,bc,mrt", CASES)
def test_tuning_keeps_the_faster_own_launches(nx, ny, store, bc, mrt, tmp_path):
    cache = str(tmp_path / "tiles.json")
    g, ref = _lattice(nx, ny, store, bc, mrt), _lattice(nx, ny, store, bc, mrt)
    L.lbm_set_two_step(ref.ctx, -1)
    entry = autotune.tune(g, store, reps=3, path=cache)
    assert entry["two_step"] == autotune.AUTO and 0 < entry["auto_ms"] < entry["ms"]
    assert g.t == 0 and _three_steps_in_one_launch(g)
    # the single-step tuner alone, on an untouched lattice and on one whose single steps were asked for
    h = _lattice(nx, ny, store, bc, mrt)
    h.autotune(reps=3)
    assert _three_steps_in_one_launch(h)
    L.lbm_set_two_step(h.ctx, -1)
    h.autotune(reps=1)
    assert not _three_steps_in_one_launch(h)
    # from the cache, and back by the call
    assert autotune.apply(h, store, cache) == f"{entry['tile']} | {autotune.AUTO}"
    assert _three_steps_in_one_launch(h)
    L.lbm_set_tile(h.ctx, 0)
    assert not _three_steps_in_one_launch(h)
    L.lbm_set_auto_launch(h.ctx)
    assert _three_steps_in_one_launch(h)
    g.step(h.t - g.t)
    ref.step(h.t)
    assert torch.equal(g.populations(), ref.populations()) and torch.equal(h.populations(), ref.populations())
    for lat in (g, h, ref):
        lat.close()


def test_choices_the_tuners_time_themselves_report_none():
    """Single steps (a lattice below the deep sweep's reach, timing, separate launches) and multi-step shapes."""
    for nx, ny, store, prepare in ((17, 17, "f32", None), (2048, 1100, "f32", None),
                                   (128, 128, "f32", lambda c: L.lbm_enable_timing(c, True)),
                                   (128, 128, "f32", lambda c: L.lbm_set_fused(c, False))):
        g = _lattice(nx, ny, store, (1, 1, 1, 1), None)
        if prepare:
            prepare(g.ctx)
        assert L.lbm_time_auto_launch(g.ctx, 2) == -1.0
        g.close()
