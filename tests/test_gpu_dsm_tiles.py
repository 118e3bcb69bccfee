"""The fused dynamic-model kernel at the edges of its tiles (32 x 16 cells in FP64), z chunks and wall layers:
nu_t against the oracle, cell by cell, within the derived rounding bound of two float64 evaluations."""
import numpy as np
import pytest

from oracle.case import SGS_DSM
from oracle import substep as S
from tests.cases import dsm_nut_check, initial_fields, make_pair, say

pytestmark = pytest.mark.gpu
PER, NOSLIP, WM = 0, 1, 2

# grids narrower than a tile, with a remainder in x, in y or both, whole tiles; the fewest planes, one plane
# more than a chunk, several chunks
CASES = [(PER, 20, 12, 10, 0), (PER, 64, 32, 6, 0), (PER, 40, 48, 64, 0),
         (NOSLIP, 8, 4, 4, 0), (NOSLIP, 40, 20, 5, 0), (NOSLIP, 96, 16, 33, 0),
         (WM, 8, 6, 4, 0), (WM, 30, 30, 7, 0), (WM, 32, 16, 6, 0), (WM, 96, 48, 37, 0),
         (NOSLIP, 40, 20, 5, 1), (NOSLIP, 32, 48, 17, 1), (WM, 8, 6, 4, 1), (WM, 30, 16, 9, 1), (WM, 64, 48, 21, 1)]


@pytest.mark.parametrize("zbc,nx,ny,nz,ybc", CASES)
def test_dynamic_model_at_tile_edges(zbc, nx, ny, nz, ybc):
    from paper_2411_09364_amd import les
    case, g, cfg = make_pair(nx, ny, nz, 3.0, 2.0, 2.0, zbc=zbc, beta=0.0 if zbc == PER or ybc else 1.3, nu=1e-3,
                             sgs=SGS_DSM, ybc=ybc)
    u, v, w = initial_fields(case, g, 11, "random")
    # long waves over the noise, so that the plane (line, box) sums of L_ij M_ij are not all clipped
    x, y, z = (np.arange(a.shape[q]) * 2.0 * np.pi / m for a, q, m in ((u, 2, nx), (u, 1, ny), (u, 0, nz)))
    X, Y, Z = x[None, None, :], y[None, :, None], z[:, None, None]
    u, v, w = (0.05 * f + np.sign(np.abs(f)) * s for f, s in
               ((u, np.sin(Y + Z) + np.cos(2 * X)), (v, np.sin(X - Z) * np.cos(Y)), (w, np.cos(X + 2 * Y))))
    st = S.initial_state(case, g, u, v, w)
    solver = les.Solver(cfg)
    solver.set_state(u, v, w)
    solver.nut()
    nut = solver.eddy_viscosity()
    solver.close()
    ok, ratio, bound = dsm_nut_check(case, g, st, nut)
    say(f"dsm {zbc} {nx}x{ny}x{nz} ybc {ybc}: worst ratio {ratio:.3f}, c_s rounding bound {bound:.1e}")
    assert np.max(np.abs(st.nut)) > 0 and ok, ratio
