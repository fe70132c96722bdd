"""pic_step, pic_sync and pic_diag on a grid of 13.5 M tiles of 8 x 8 cells and
four species, whose sort plan and field blocks together are more than 2^32
threads on one axis.

Fields zero at the start, so E after the step is -dt J in every cell (one
rounding), and each particle streams freely for the step; the sections are
those of the cells that pic_sync writes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_step_on_millions_of_tiles():
    import torch
    from paper_2501_14795_amd import Sim, _lib
    N, T, DX, DT = 29376, 8, 0.1, 0.07
    rng = np.random.default_rng(11)
    species = []
    for k in range(4):
        n = 20000 + 64 * k
        tile = np.sort(rng.integers(0, (N // T) ** 2, n))
        tile[:40], tile[-40:] = 0, (N // T) ** 2 - 1     # the first and the last tile, whose particles cross the seam
        st = {"ix": (tile % (N // T) * T + rng.integers(0, T, n)).astype(np.int32),
              "iy": (tile // (N // T) * T + rng.integers(0, T, n)).astype(np.int32)}
        for f in ("x", "y"):
            st[f] = rng.uniform(0, 0.999, n).astype(np.float32)
        for f in ("ux", "uy", "uz"):
            st[f] = rng.normal(0, 0.8, n).astype(np.float32)
        species.append(st)
    sim = Sim(N, N, DX, DX, DT, T, [(-1.0, -0.5, st) for st in species])
    sim.step()
    sim.sync()
    assert sim.check() == 0
    E, J = sim.fields[:3], sim.fields[6:]
    assert float(J.abs().amax()) > 0 and float(J[:, -1, -1].abs().amax()) > 0
    for c in range(3):   # one plane at a time
        assert float((E[c] + np.float32(DT) * J[c]).abs().amax()) <= 2e-7 * float(J[c].abs().amax())
    for k, st in enumerate(species):
        g = sim.state(k)
        t = g["iy"].astype(np.int64) // T * (N // T) + g["ix"] // T
        assert (np.diff(t) >= 0).all()
        off = sim.tile_offsets(k)
        assert np.array_equal(off, np.searchsorted(t, np.arange((N // T) ** 2 + 1)))
        gamma = np.sqrt(1 + sum(st[u].astype(np.float64) ** 2 for u in ("ux", "uy", "uz")))
        X = (st["ix"] + st["x"].astype(np.float64) + st["ux"] / gamma * (DT / DX)) % N
        Y = (st["iy"] + st["y"].astype(np.float64) + st["uy"] / gamma * (DT / DX)) % N
        want, got = np.lexsort((st["uy"], st["ux"])), np.lexsort((g["uy"], g["ux"]))
        for a, b, i in ((X, g["ix"] + g["x"].astype(np.float64), "x"), (Y, g["iy"] + g["y"].astype(np.float64), "y")):
            d = np.abs(a[want] - b[got])
            assert np.minimum(d, N - d).max() < 1e-6, (k, i)
    d = sim.diag(_lib.PIC_DIAG_ENERGY)
    assert d.u_e > 0 and all(d.u_k[k] > 0 for k in range(4))
    sim.close()
