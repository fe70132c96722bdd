"""The sort plan's inputs where they change: the new sections counted by every
plan block (up to 256 tiles), from the recount's prefixes (beyond), and the
leavers listed by direction, on axes of one, two and three tiles (where
neighbours coincide or wrap onto each other), with a hot plasma (a third of
the particles leave their tile in a step on 8 x 8 tiles) and empty tiles.
pic_sort bit for bit against the oracle's canonical sort, three steps in a row, and pic_step
equal to the separate calls."""
import numpy as np
import pytest

import pic_workloads as pw
from _parity import flush, sort_replay, species_states

pytestmark = pytest.mark.gpu

DX = DY = 0.1
DT = 0.07


@pytest.mark.parametrize("tx,ty,tile,ppc,box", [
    (16, 16, 8, (2, 2), None),          # 256 tiles: the last the plan counts itself
    (257, 1, 8, (2, 2), None),          # 257: one more, one tile high
    (1, 1, 16, (4, 4), None),
    (2, 1, 8, (5, 3), None),
    (2, 2, 8, (3, 3), None),
    (3, 2, 16, (3, 5), None),
    (3, 3, 32, (2, 2), (20, 50, 0, 96)),   # most tiles partly or wholly empty
    (40, 13, 8, (1, 1), None),
])
def test_plan_lists(tx, ty, tile, ppc, box):
    from paper_2501_14795_amd import Sim
    nx, ny = tx * tile, ty * tile
    specs = [pw.SpeciesSpec(-1.0, ppc, (1.5, 1.5, 0.2), (0.5, -0.7, 0.0)),
             pw.SpeciesSpec(-1.0, (1, 2), (0.3, 2.5, 0.2), (-0.5, 0.0, 0.0))]
    states = species_states(nx, ny, tile, specs, 11, cell_box=box)
    E, B = pw.random_fields(nx, ny, 0.1, 3)
    sims = [Sim(nx, ny, DX, DY, DT, tile, [(s.qm, s.q, st) for s, st in zip(specs, states)], E=E, B=B) for _ in range(2)]
    for _ in range(3):
        sims[0].push_deposit()
        sort_replay(sims[0], specs, tile)
        sims[0].field_advance()
        sims[1].step()
    for k in range(2):
        a, b = sims[0].state(k), sims[1].state(k)
        for f in a:
            assert np.array_equal(a[f], b[f]), f
        assert np.array_equal(sims[0].tile_offsets(k), sims[1].tile_offsets(k))
    fa, fb = sims[0].field_arrays(), sims[1].field_arrays()
    assert all(np.array_equal(fa[c], fb[c]) for c in fa)
    assert all(s.check() == 0 for s in sims)
    flush(f"{tx}x{ty} tiles of {tile}: {[st['ix'].size for st in states]} particles, three sorts bit-exact")
    for s in sims:
        s.close()
