"""Ensembles large enough for their three-step sweep to march its members, against single steps: every stored
population the same bits, with the work list in runs (state beyond the L2s) and in stretches (state within
them), at widths around the last strip's overlap and with members that stay in tiles."""
import numpy as np
import pytest

from paper_2005_08674_amd import lbm as L

pytestmark = pytest.mark.gpu

MARCH_TILES, L2_BYTES = 1024, 32 << 20  # the library's limits, from which members march and lists go in runs
ESIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
# below the march's least size, at it, around one, two and three strips, and several chunks
SIZES = [(64, 20), (95, 71), (96, 48), (96, 72), (97, 73), (144, 100), (145, 131), (159, 119), (160, 120), (161, 121),
         (208, 210), (209, 201), (225, 420), (300, 64), (500, 260)]


def _members(store, copies, extra):
    from paper_2005_08674_amd.ensemble import member_params
    sizes = SIZES * copies + extra
    members, fields = [], []
    for k, (nx, ny) in enumerate(sizes):
        u = (0.04, -0.02) if k % 2 else (0.0, 0.0)
        members.append(member_params(nx, ny, 0.57, store=store, ubase=u, mrt=(1.6, 1.4, 1.8) if k % 3 == 2 else None))
        r = np.random.default_rng(nx * 7 + ny + k)
        fields.append(tuple(1e-3 * r.standard_normal((ny, nx)) + c for c in (0.0, *u)))
    tiles = {ty: sum(-(-nx // 64) * -(-ny // ty) for nx, ny in sizes) for ty in (8, 12)}
    state = sum(2 * 9 * ny * -(-nx * ESIZE[store] // 256) * 256 for nx, ny in sizes)
    return members, fields, tiles, state


@pytest.mark.parametrize("store,copies,extra,runs", [
    ("f64", 2, [(512, 400)], True), ("f32", 2, [(512, 400)], True), ("f16", 1, [(512, 400), (320, 200)], False),
    ("bf16", 3, [(512, 512)], True)])
def test_marched_ensemble_equals_single_steps(store, copies, extra, runs):
    from paper_2005_08674_amd.ensemble import Ensemble
    members, fields, tiles, state = _members(store, copies, extra)
    assert min(tiles.values()) >= MARCH_TILES, tiles
    assert state > 1.05 * L2_BYTES if runs else state < 0.95 * L2_BYTES, state
    ref = Ensemble(members, fields)
    ref.step(9)
    want = [ref.populations(m) for m in range(len(members))]
    ref.close()
    seen = 0
    for shape in range(L.lbm_two_step_count()):
        name = L.lbm_two_step_describe(shape)
        if not name.startswith(("3step:64x12", "3step:64x8")) or "+march" in name:
            continue
        e = Ensemble(members, fields)
        e.set_two_step(shape)
        e.step(3)
        e.step_graph(6)
        for m in range(len(members)):
            assert np.array_equal(e.populations(m), want[m]), (name, members[m].nx, members[m].ny)
        e.close()
        seen += 1
    assert seen >= 3
