"""The push's lists of leavers by direction where a wavefront finds more of
them than its buffer of 64 entries holds (the rest is read back), for one
species and for a later one whose entries start in the middle of it or beyond:
with 4, 8 and 16 wavefronts per tile.  pic_sort bit for bit against the
oracle's canonical sort."""
import numpy as np
import pytest

import pic_workloads as pw
from _parity import flush, sort_replay, species_states

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tx,ty,tile,ppc", [
    (17, 17, 8, ((6, 6), (6, 6))),                      # 4 wavefronts, about 190 leavers each
    (17, 17, 8, ((2, 2), (4, 4), (1, 1), (2, 3))),      # entries of all four species in one buffer
    (17, 16, 32, ((3, 3),)),                            # 8 wavefronts
    (16, 16, 8, ((12, 12), (2, 2))),                    # 16 wavefronts
])
def test_many_leavers(tx, ty, tile, ppc):
    from paper_2501_14795_amd import Sim
    nx, ny = tx * tile, ty * tile
    specs = [pw.SpeciesSpec(-1.0, p, (1.5, 1.5, 0.2), ((0.5, -0.7, 0.0), (-0.5, 0.3, 0.0))[k % 2])
             for k, p in enumerate(ppc)]
    states = species_states(nx, ny, tile, specs, 13)
    sim = Sim(nx, ny, 0.1, 0.1, 0.07, tile, [(s.qm, s.q, st) for s, st in zip(specs, states)])
    for _ in range(2):
        off = sim.tile_offsets(0)
        sim.push_deposit()
        pre = sort_replay(sim, specs, tile)
        sim.field_advance()
    t = pre[0]["iy"] // tile * tx + pre[0]["ix"] // tile
    left = (t != np.repeat(np.arange(tx * ty), np.diff(off))).sum() / (tx * ty)
    flush(f"{tx}x{ty} tiles of {tile}: {left:.0f} leavers a tile, two sorts bit-exact")
    sim.close()
