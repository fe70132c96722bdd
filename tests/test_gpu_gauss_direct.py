"""The direct (Hartley transform) solve of pic_solve_gauss at grid sizes
around its 32 x 32 tiles and 32-term stages -- edges of 8, remainders of 8, 16
and 24, one tile, long and thin -- against the oracle's FFT projection.

The solve satisfies ||r|| <= 1e-12 ||r0|| in FP64 and stores FP32: E and B
within one unit of FP32 rounding of max|F| of the oracle's (2^-23; the
correction and the stored result are each rounded once)."""
import numpy as np
import pytest

import oracle
import pic_workloads as pw
from _parity import flush, rel_err, species_states

pytestmark = pytest.mark.gpu

DX, DY, DT = 0.1, 0.12, 0.06


@pytest.mark.parametrize("nx,ny,tile", [(8, 8, 8), (40, 24, 8), (56, 72, 8), (32, 32, 32), (264, 16, 8), (16, 1032, 8),
                                        (96, 160, 32)])
def test_direct_solve_matches_oracle(nx, ny, tile):
    from paper_2501_14795_amd import Sim
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
    out = sim.solve_gauss()
    f = sim.field_arrays()
    eE, eB = rel_err(f["E"], Eo), rel_err(f["B"], Bo)
    flush(f"{nx}x{ny}: {list(out.iterations)} iterations, residuals {list(out.residual)}, E {eE:.2e} B {eB:.2e}")
    assert eE <= 2.0 ** -23 and eB <= 2.0 ** -23
    assert max(out.residual) <= 1e-12
    assert max(out.iterations) <= 3   # direct solves, not conjugate gradients
    sim.close()
