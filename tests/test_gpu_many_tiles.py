"""Oracle replays of every deposit, shape, filter and cadence on 17 x 17
tiles: above 256 tiles a simulation is pushed by four wavefronts per tile
(eight for 32 x 32 tiles) instead of sixteen, and its sort plan takes the new
sections from the recount.

Each step starts from the GPU's own state: positions within 1e-5 cells,
momenta within 1e-5 of max|u|, J within 1e-5 of max|J|, every sort bit-exact
(the tolerances of the other replays)."""
import pytest

import pic_workloads as pw
from _parity import flush, make_pair, oracle_from_gpu, particle_errors, rel_err, sort_replay, species_states

pytestmark = pytest.mark.gpu

DX = DY = 0.1
DT = 0.07


@pytest.mark.parametrize("tile,nspecies,options", [
    (8, 2, {}),
    (16, 1, {}),
    (32, 1, {}),
    (8, 1, {"esirkepov": True}),
    (16, 2, {"esirkepov": True, "j_filter": 2}),
    (32, 1, {"esirkepov": True}),
    (8, 1, {"quadratic": True}),
    (16, 1, {"quadratic": True}),
    (32, 2, {"quadratic": True, "j_filter": 1}),
    (8, 1, {"sort_every": 2}),
    (16, 1, {"sort_every": 2}),
    (16, 1, {"sort_every": 4}),
    (16, 1, {"sort_every": 2, "esirkepov": True}),
    (32, 1, {"sort_every": 2}),
    (32, 1, {"sort_every": 4}),
    (16, 1, {"motion_sort": True}),
])
def test_replay_above_256_tiles(tile, nspecies, options):
    nx = ny = 17 * tile
    ppc = (2, 2) if tile < 32 else (1, 2)
    specs = [pw.SpeciesSpec(-1.0, ppc, (0.3, 0.3, 0.2), ((0.5, -0.4, 0.1), (-0.5, 0.3, 0.2))[k]) for k in range(nspecies)]
    states = species_states(nx, ny, tile, specs, 23)
    E, B = pw.random_fields(nx, ny, 0.05, 23)
    sim, _ = make_pair(nx, ny, DX, DY, DT, tile, specs, states, E, B, **options)
    every = options.get("sort_every", 1)
    worst = [0.0, 0.0, 0.0]
    for step in range(2 * every):
        ref = oracle_from_gpu(sim, specs, DX, DY, DT)
        for k in ("esirkepov", "quadratic", "j_filter"):
            setattr(ref, k, options.get(k, getattr(ref, k)))
        ref.push_deposit()
        sim.push_deposit()
        assert sim.check() == 0
        for k in range(nspecies):
            pos, du = particle_errors(sim.state(k), ref.species[k], nx, ny)
            worst[0], worst[1] = max(worst[0], pos), max(worst[1], du)
        worst[2] = max(worst[2], rel_err(sim.field_arrays()["J"], ref.J))
        if step % every == every - 1:
            if options.get("motion_sort"):
                sim.sort()   # its order is its own; compared by the next replay through the particles' values
                assert sim.check() == 0
            else:
                sort_replay(sim, specs, tile)
        sim.field_advance()
    flush(f"T{tile} x{nspecies} {options}: pos {worst[0]:.2e} u {worst[1]:.2e} J {worst[2]:.2e}")
    assert max(worst) < 1e-5
    sim.close()
