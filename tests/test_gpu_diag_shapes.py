"""pic_diag over particle layouts: the charge is summed in LDS tile section
by tile section (sections of fewer than 128 particles straight into the grid),
a block's range of slots spanning one tile's part or many tiles.

Against the oracle's node charge and numpy's FP64 sums on the state read back
from the GPU: both sides are FP64 and differ in the order of the sums only
(n eps of the largest term: 1e-12 relative bounds it for every case here)."""
import numpy as np
import pytest

import oracle
import pic_workloads as pw
from _parity import flush, species_states

pytestmark = pytest.mark.gpu

DX, DT = 0.1, 0.07

# (nx, ny, tile, ppc, cell box or None, quadratic, sort_every, unsorted pushes)
CASES = [
    (24, 40, 8, (1, 1), None, False, 1, 0),            # 64 particles a section: direct
    (64, 48, 16, (1, 1), None, False, 1, 1),           # 256: LDS; one push past the sort
    (96, 64, 32, (5, 3), None, True, 1, 1),            # odd sections, the wider shape
    (256, 256, 8, (8, 8), (40, 56, 80, 90), False, 1, 0),   # all particles in few of 1,024 tiles
    (64, 64, 16, (4, 4), None, False, 4, 4),           # strayed up to four cells
    (8, 8, 8, (1, 1), (2, 4, 3, 4), False, 1, 0),      # two particles, one tile
    (160, 32, 32, (16, 16), (0, 33, 0, 32), True, 1, 0),    # a full tile, a sliver, empty tiles
]


@pytest.mark.parametrize("nx,ny,tile,ppc,box,quad,every,pushes", CASES)
def test_diag_matches_fp64(nx, ny, tile, ppc, box, quad, every, pushes):
    from paper_2501_14795_amd import Sim, _lib
    spec = pw.SpeciesSpec(-1.0, ppc, (0.3, 0.3, 0.3), (0.2, -0.3, 0.0))
    st = species_states(nx, ny, tile, [spec], 5, cell_box=box)[0]
    rng = np.random.default_rng(nx + tile)
    st["x"] = np.minimum(rng.uniform(0, 1, st["x"].size), 0.9999).astype(np.float32)
    st["y"] = np.minimum(rng.uniform(0, 1, st["y"].size), 0.9999).astype(np.float32)
    E, B = pw.random_fields(nx, ny, 0.1, 5)
    sim = Sim(nx, ny, DX, DX, DT, tile, [(spec.qm, spec.q, st)], E=E, B=B, quadratic=quad, sort_every=every)
    for _ in range(pushes):
        sim.push_deposit()
    d = sim.diag(_lib.PIC_DIAG_ENERGY | _lib.PIC_DIAG_GAUSS)
    k = sim.diag(_lib.PIC_DIAG_ENERGY)
    g, f = sim.state(0), sim.field_arrays()
    Ed, Bd = f["E"].astype(np.float64), f["B"].astype(np.float64)
    rho = oracle.rho(nx, ny, spec.q, g["ix"], g["iy"], g["x"], g["y"], **({"quadratic": True} if quad else {}))
    u2 = sum(g[c].astype(np.float64) ** 2 for c in ("ux", "uy", "uz"))
    want = {"u_e": 0.5 * DX * DX * (Ed ** 2).sum(), "u_b": 0.5 * DX * DX * (Bd ** 2).sum(),
            "u_k": DX * DX * (spec.q / spec.qm) * (u2 / (np.sqrt(1 + u2) + 1)).sum(),
            "gauss_max": np.abs(oracle.div_e(nx, ny, DX, DX, Ed) - (rho - spec.q * g["x"].size / (nx * ny))).max(),
            "divb_max": np.abs(oracle.div_b(nx, ny, DX, DX, Bd)).max()}
    for name, w in want.items():
        for o in (d,) if name.endswith("max") else (d, k):
            got = o.u_k[0] if name == "u_k" else getattr(o, name)
            assert abs(got - w) <= 1e-12 * abs(w), (name, got, w)
    flush(f"{nx}x{ny} T{tile}, {g['x'].size} particles: {want}")
    assert sim.check() == 0
    sim.close()


def test_diag_reports_nan():
    """A NaN in one field value reaches the residuals' maxima."""
    from paper_2501_14795_amd import Sim, _lib
    spec = pw.SpeciesSpec(-1.0, (2, 2), (0.1, 0.1, 0.1), (0.0, 0.0, 0.0))
    st = species_states(64, 512, 16, [spec], 5)[0]
    sim = Sim(64, 512, DX, DX, DT, 16, [(spec.qm, spec.q, st)])
    sim.fields[0, 300, 7] = float("nan")
    d = sim.diag(_lib.PIC_DIAG_GAUSS | _lib.PIC_DIAG_ENERGY)
    assert np.isnan(d.gauss_max) and np.isnan(d.u_e) and d.divb_max == 0.0 and d.u_b == 0.0
    sim.close()
