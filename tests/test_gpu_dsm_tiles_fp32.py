"""The fused dynamic-model kernel in FP32 (periodic boxes with explicit viscous terms: 32 x 8 tiles, three blocks per
CU) at the edges of its tiles and z chunks: nu_t against the oracle, cell by cell, within the derived rounding bound
of two evaluations of the model, taken with FP32's unit roundoff but for the plane sums, which both sides form in
FP64; |S| alone, nu_t over its coefficient, within the bound of the strain, a few roundings.  The input is exact in
FP32, and the ghosts are copies."""
import numpy as np
import pytest

from oracle import substep as S
from oracle.case import SGS_DSM
from tests import dsm_bound
from tests.cases import dsm_nut_check, make_pair, round32, say

pytestmark = pytest.mark.gpu

# narrower than a tile, a remainder in x, in y, in both, whole tiles; the fewest planes, odd counts, several chunks
GRIDS = [(8, 6, 4), (20, 12, 5), (32, 8, 15), (40, 10, 16), (64, 20, 30), (96, 40, 48), (30, 24, 64)]


def fp32_case(nx, ny, nz, monkeypatch):
    """A long wave per component under noise, of the sign whose c_s is not clipped (L_ij M_ij is odd in u)."""
    depth = dsm_bound.plane_sum_depth
    monkeypatch.setattr(dsm_bound, "U", 2.0 ** -24)
    monkeypatch.setattr(dsm_bound, "plane_sum_depth", lambda case, g: depth(case, g) * 2.0 ** -29)
    case, g, cfg = make_pair(nx, ny, nz, 3.0 * nx / 32, 2.0 * ny / 20, 2.0 * nz / 20, nu=1e-3, sgs=SGS_DSM, precision=1)
    r = np.random.Generator(np.random.PCG64(nx + ny + nz))
    X, Y, Z = (2.0 * np.pi * np.arange(n).reshape(s) / n for n, s in ((nx, (1, 1, -1)), (ny, (1, -1, 1)), (nz, (-1, 1, 1))))
    waves = (np.sin(Y + 0.3) * np.cos(Z), np.sin(Z + 0.7) * np.cos(X), np.sin(X + 0.2) * np.cos(Y))
    fields = []
    for f in waves:
        a = np.zeros((nz + 2, ny, nx))
        a[1:nz + 1] = f + r.standard_normal((nz, ny, nx))
        a[0], a[nz + 1] = a[nz], a[1]
        fields.append(a)
    fields = round32(*fields)
    st = S.initial_state(case, g, *fields)
    if np.max(st.nut) == 0.0:
        fields = tuple(-a for a in fields)
        st = S.initial_state(case, g, *fields)
    return case, g, cfg, fields, st


@pytest.mark.parametrize("nx,ny,nz", GRIDS)
def test_dynamic_model_at_tile_edges_fp32(nx, ny, nz, monkeypatch):
    from paper_2411_09364_amd import les
    case, g, cfg, fields, st = fp32_case(nx, ny, nz, monkeypatch)
    solver = les.Solver(cfg)
    solver.set_state(*fields)
    solver.nut()
    nut, cs = solver.eddy_viscosity(), solver.coefficient()
    solver.close()
    # |S| of two evaluations and the roundings of its product with the coefficient
    I = slice(1, nz + 1)
    s = dsm_bound.strain_magnitude(dsm_bound.centre_strain(g, *(dsm_bound.D(a) for a in (st.u, st.v, st.w))))
    got = nut[I] / (cs * g.delta() ** 2)[:, None, None]
    worst = np.max(np.abs(got - s.v) / (2.0 * s.e + 4.0 * dsm_bound.U * s.v))
    assert np.max(s.e) < 1e-5 * np.max(s.v) and worst <= 1.0, worst
    ok, ratio, bound = dsm_nut_check(case, g, st, nut)
    say(f"dsm fp32 {nx}x{ny}x{nz}: |S| ratio {worst:.3f}, nu_t {ratio:.3f}, rounding bound {bound:.1e} of the largest nu_t")
    assert np.max(st.nut) > 0 and bound < 0.1
    assert ok, ratio
