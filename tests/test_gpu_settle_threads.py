"""pic_sync with every number of threads per tile that its launch can choose
(16 to 1,024 by the particles a tile holds on average), several tiles side by
side in a block and a remainder of them, alone and in a batch: the caller's
cell arrays, overwritten before the call, hold every particle's cell again."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _load(ntx, nty, tile, mean, seed):
    """About `mean` particles a tile (0 to 2 mean), grouped by tile."""
    rng = np.random.default_rng(seed)
    k = rng.integers(0, 2 * mean + 1, ntx * nty)
    t = np.repeat(np.arange(ntx * nty), k)
    st = {"ix": (t % ntx * tile + rng.integers(0, tile, t.size)).astype(np.int32),
          "iy": (t // ntx * tile + rng.integers(0, tile, t.size)).astype(np.int32)}
    for f in ("x", "y"):
        st[f] = rng.uniform(0, 0.999, t.size).astype(np.float32)
    for f in ("ux", "uy", "uz"):
        st[f] = np.zeros(t.size, np.float32)
    return st


@pytest.mark.parametrize("mean", [1, 100, 200, 400, 800, 1600, 6000])
def test_sync_writes_the_cells(mean):
    import torch
    from paper_2501_14795_amd import Sim, Batch
    from paper_2501_14795_amd.sim import pack_cells
    shapes = [(3, 5, 8), (2, 7, 8)]
    loads = [[_load(ntx, nty, T, mean, 10 * k + s) for s in range(2)] for k, (ntx, nty, T) in enumerate(shapes)]
    members = [dict(nx=ntx * T, ny=nty * T, dx=0.1, dy=0.1, dt=0.07, species=[(-1.0, -0.1, st) for st in sp])
               for (ntx, nty, T), sp in zip(shapes, loads)]
    sims = [Sim(m["nx"], m["ny"], 0.1, 0.1, 0.07, 8, m["species"]) for m in members]
    batch = Batch(members, 8)

    def spoil(view):
        for p in view.particles:
            p["cell"].fill_(-7)

    for view in sims + [batch[0], batch[1]]:
        spoil(view)
    torch.cuda.synchronize()
    for s in sims:
        s.sync()
    batch.sync()
    torch.cuda.synchronize()
    for view, sp in zip(sims + [batch[0], batch[1]], loads + loads):
        for p, st in zip(view.particles, sp):
            assert np.array_equal(p["cell"].cpu().numpy(), pack_cells(st["ix"], st["iy"]))
    for s in sims:
        s.close()
    batch.close()
