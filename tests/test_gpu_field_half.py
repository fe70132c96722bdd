"""pic_step's field half in one launch works on regions of 64 x 8 cells and
computes E one cell beyond each from the push's edge strips; above 2^21 cells
it is two launches.  Grids whose regions end inside, at and past 64 columns, a
single region that is its own neighbour, every tile edge and halo pad, the
filter (J read, not folded), many small members of a batch, and one grid on
each side of the limit: E, B and J bit for bit those of the separate calls
(three in-place launches)."""
import numpy as np
import pytest

import pic_workloads as pw
from _parity import flush, species_states

pytestmark = pytest.mark.gpu

DX, DY, DT = 0.1, 0.12, 0.06


@pytest.mark.parametrize("nx,ny,tile,options", [
    (8, 8, 8, {}),
    (56, 24, 8, {}),
    (64, 8, 8, {"sort_every": 2}),
    (72, 16, 8, {"quadratic": True}),
    (128, 48, 16, {"j_filter": 1}),
    (144, 80, 16, {"sort_every": 4}),
    (96, 64, 32, {"quadratic": True}),
    (160, 32, 32, {"esirkepov": True}),
    (2048, 1024, 32, {}),
    (2080, 1024, 32, {}),
    (1408, 1504, 32, {"j_filter": 2}),
])
def test_step_equals_the_separate_calls(nx, ny, tile, options):
    from paper_2501_14795_amd import Batch, Sim
    spec = pw.SpeciesSpec(-1.0, (1, 1), (0.4, 0.4, 0.4), (0.1, 0.2, 0.0))
    st = species_states(nx, ny, tile, [spec], 17)[0]
    E, B = pw.random_fields(nx, ny, 0.2, 9)
    rng = np.random.default_rng(3)
    E += rng.normal(0, 0.02, E.shape).astype(np.float32)
    B += rng.normal(0, 0.02, B.shape).astype(np.float32)
    args = (nx, ny, DX, DY, DT, tile, [(spec.qm, spec.q, st)])
    one, apart = Sim(*args, E=E, B=B, **options), Sim(*args, E=E, B=B, **options)
    small = nx * ny <= 1 << 16
    member = {"nx": nx, "ny": ny, "dx": DX, "dy": DY, "dt": DT, "species": args[6], "E": E, "B": B}
    batch = Batch([member] * 3, tile, **options) if small else None
    every = options.get("sort_every", 1)
    for k in range(4):
        one.step()
        if batch:
            batch.step()
        apart.push_deposit()
        if (k + 1) % every == 0:
            apart.sort()
        apart.field_advance()
        want = apart.field_arrays()
        for s in [one] + ([batch[1], batch[2]] if batch else []):
            got = s.field_arrays()
            for c in want:
                assert np.array_equal(got[c], want[c]), (k, c)
    assert one.check() == 0 and apart.check() == 0
    flush(f"{nx}x{ny} T{tile} {options}: fields equal over 4 steps")
    one.close()
    apart.close()
    if batch:
        batch.close()
