"""Window moves whose new particles' first slots, those after the existing
particles, already lie in their own tile's new section: a species that starts
empty, more plasma coming in than leaves (a vacuum column leaving, a denser
column entering), with the origin in the first and in the last tile column and
on a grid of a single tile row.  Such a particle stays where it was appended:
its slot is no hole.

The expected layout is the oracle's canonical sort, in array columns, of the
state before the move with the origin column's particles removed and the new
ones appended; everything is compared bit for bit."""
import numpy as np
import pytest

import oracle
import pic_workloads as pw

pytestmark = pytest.mark.gpu

ARRAYS = ("ix", "iy", "x", "y", "ux", "uy", "uz")


def _load(nx, ny, tile, per_axis, seed, box):
    return pw.species_state(nx, ny, tile, pw.SpeciesSpec(-1.0, per_axis, (0.1,) * 3, (0.0, 0.0, 0.0)), seed, 0, cell_box=box)


def _none():
    return {a: np.zeros(0, np.int32 if a in ("ix", "iy") else np.float32) for a in ARRAYS}


@pytest.mark.parametrize("nx,ny,tile,start,new,first", [
    (64, 48, 16, None, (4, 4), 0),            # a species that starts empty
    (64, 48, 16, None, (4, 4), 63),           # the same, origin in the last tile column
    (64, 48, 16, (1, 63), (2, 4), 0),         # a vacuum column leaves, plasma comes in
    (64, 48, 16, (0, 63), (2, 4), 63),        # the same in the last tile column
    (64, 16, 16, (0, 64), (5, 5), 0),         # one tile row, fewer leave than come in
    (64, 16, 16, (0, 64), (5, 5), 63),
    (160, 136, 8, (0, 160), (5, 5), 159),     # more than 256 tiles
    (96, 64, 32, (0, 96), (1, 1), 95),        # fewer come in than leave
])
def test_injected_into_their_own_section(nx, ny, tile, start, new, first):
    from paper_2501_14795_amd import Sim
    st = _none() if start is None else _load(nx, ny, tile, (2, 2), 3, (start[0], start[1], 0, ny))
    n0 = st["ix"].size
    sim = Sim(nx, ny, 0.1, 0.1, 0.07, tile, [(-1.0, -0.25, st)], moving_window=True, capacity=[n0 + 200 * ny])
    # the window origin `first`: the state loaded with it
    state = sim.get_state()
    state["window_origin"] = first
    sim.set_state(state)
    for move in range(3):
        origin = sim.window_origin()
        assert origin == (first + move) % nx
        pre = sim.state(0)
        inject = _load(nx, ny, tile, new, 50 + move, (nx - 1, nx, 0, ny))
        sim.move_window([inject])
        k = inject["ix"].size
        cat = {a: np.r_[pre[a], inject[a]] for a in ARRAYS}
        cat["ix"][pre["ix"].size:] = origin
        removed = np.r_[pre["ix"] == origin, np.zeros(k, bool)]
        off, src = oracle.sort_canonical(nx, ny, tile, cat["ix"], cat["iy"], removed=removed)
        assert sim.counts()[0] == src.size
        got = sim.state(0)
        for a in ARRAYS:
            assert np.array_equal(got[a], cat[a][src]), (move, a)
        assert np.array_equal(sim.tile_offsets(0), off)
    sim.step()
    assert sim.check() == 0
    sim.close()
