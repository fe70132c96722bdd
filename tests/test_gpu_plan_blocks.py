"""pic_step's sort plan and field half, in one launch with four tiles per plan
block, with ten (from 2,560 tile sections on), or in two (from 16,384; a batch
from 8,192): particles, sections and fields bit for bit those of the separate
calls (pic_push_deposit, pic_sort, pic_field_advance)."""
import numpy as np
import pytest

import pic_workloads as pw
from _parity import PARTICLE_ARRAYS, species_states

pytestmark = pytest.mark.gpu

DX, DY, DT = 0.1, 0.12, 0.06


def _load(nx, ny, tile, nspecies):
    specs = [pw.SpeciesSpec(-1.0, (1, 1), (0.4, 0.4, 0.4), (0.3 - 0.5 * k, 0.2, 0.0)) for k in range(nspecies)]
    E, B = pw.random_fields(nx, ny, 0.2, 9)
    return [(s.qm, s.q, st) for s, st in zip(specs, species_states(nx, ny, tile, specs, 17))], E, B


def _equal(a, b, nspecies, step):
    fa, fb = a.field_arrays(), b.field_arrays()
    for c in fa:
        assert np.array_equal(fa[c], fb[c]), (step, c)
    for k in range(nspecies):
        assert np.array_equal(a.tile_offsets(k), b.tile_offsets(k)), step
        pa, pb = a.state(k), b.state(k)
        for name in PARTICLE_ARRAYS:
            assert np.array_equal(pa[name], pb[name]), (step, k, name)


# tiles: 2,550; 2,601 (a last block of one); 2 x 1,296; 16,383; 16,384; 32,940 (2.1 M cells: E and B apart); 2 x 8,281
@pytest.mark.parametrize("ntx,nty,nspecies", [(50, 51, 1), (51, 51, 1), (36, 36, 2), (129, 127, 1), (128, 128, 1), (183, 180, 1),
                                              (91, 91, 2)])
def test_step_equals_the_separate_calls(ntx, nty, nspecies):
    from paper_2501_14795_amd import Sim
    nx, ny = 8 * ntx, 8 * nty
    species, E, B = _load(nx, ny, 8, nspecies)
    one, apart = (Sim(nx, ny, DX, DY, DT, 8, species, E=E, B=B) for _ in range(2))
    for step in range(3):
        one.step()
        apart.push_deposit()
        apart.sort()
        apart.field_advance()
        _equal(one, apart, nspecies, step)
    assert one.check() == 0 and apart.check() == 0
    one.close()
    apart.close()


# sections in groups of four: 2 x 4,092 (below the line), 2 x 4,096 (on it)
@pytest.mark.parametrize("ntx,nty", [(62, 66), (64, 64)])
def test_batch_step_equals_the_separate_calls(ntx, nty):
    from paper_2501_14795_amd import Batch, Sim
    nx, ny = 8 * ntx, 8 * nty
    species, E, B = _load(nx, ny, 8, 1)
    batch = Batch([dict(nx=nx, ny=ny, dx=DX, dy=DY, dt=DT, species=species, E=E, B=B)] * 2, 8)
    apart = Sim(nx, ny, DX, DY, DT, 8, species, E=E, B=B)
    for step in range(2):
        batch.step()
        apart.push_deposit()
        apart.sort()
        apart.field_advance()
        _equal(batch[1], apart, 1, step)
    assert batch.check() == 0 and apart.check() == 0
    batch.close()
    apart.close()
