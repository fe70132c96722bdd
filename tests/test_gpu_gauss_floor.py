"""The direct solve of pic_solve_gauss with a tolerance below what FP64 can
reach: it ends after the few solves that still gain something, reports
PIC_ENOCONV with the residual it reached (round-off: well under 1e-14 of the
first), and E and B are the oracle's to FP32 rounding all the same."""
import ctypes

import numpy as np
import pytest

import oracle
import pic_workloads as pw
from _parity import flush, rel_err, species_states

pytestmark = pytest.mark.gpu

DX, DY, DT = 0.1, 0.12, 0.06


@pytest.mark.parametrize("nx,ny,tile", [(8, 8, 8), (40, 24, 8), (264, 16, 8), (128, 160, 32)])
@pytest.mark.parametrize("tol", [1e-18, 1e-200])
def test_unreachable_tolerance_ends_early(nx, ny, tile, tol):
    from paper_2501_14795_amd import Sim, _lib
    spec = pw.SpeciesSpec(-1.0, (3, 2), (0.05, 0.05, 0.05), (0.0, 0.0, 0.0))
    st = species_states(nx, ny, tile, [spec], 7)[0]
    rng = np.random.default_rng(nx * ny)
    for f in ("x", "y"):
        st[f] = np.minimum(rng.uniform(0, 1, st[f].size), 0.9999).astype(np.float32)
    E, B = pw.random_fields(nx, ny, 0.2, 3)
    B[0] += rng.normal(0, 0.05, (ny, nx)).astype(np.float32)
    rho = oracle.rho(nx, ny, spec.q, st["ix"], st["iy"], st["x"], st["y"])
    Eo, Bo = E.astype(np.float64), B.astype(np.float64)
    oracle.solve_gauss(nx, ny, DX, DY, Eo, Bo, rho)
    sim = Sim(nx, ny, DX, DY, DT, tile, [(spec.qm, spec.q, st)], E=E, B=B)
    out = _lib.pic_gauss_out()
    rc = _lib.load().pic_solve_gauss_noalloc(ctypes.c_void_p(sim.handle), tol, 0, ctypes.byref(out), ctypes.c_void_p(sim.s))
    flush(f"{nx}x{ny} tol {tol}: rc {rc}, {list(out.iterations)} solves, residuals {list(out.residual)}")
    # (a residual of exactly zero is below any tolerance)
    assert rc == _lib.PIC_ENOCONV or (rc == 0 and max(out.residual) <= tol)
    assert 1 <= max(out.iterations) <= 8
    assert max(out.residual) <= 1e-14
    f = sim.field_arrays()
    assert rel_err(f["E"], Eo) <= 2.0 ** -23 and rel_err(f["B"], Bo) <= 2.0 ** -23
    sim.close()
