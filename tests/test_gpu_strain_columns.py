"""|S| of the static models at the edges of its blocks (32 x 8 columns of up to four planes) and of the ghost rules:
remainders in x, y and z, grids of one to four planes a thread, walls, wall models and ducts; nu_t against the
oracle.  Tolerance 1e-12 of the largest nu_t: |S| is a sum of some 40 terms of velocity differences, each rounded
once (40 u = 4.4e-15), over differences that lose at most the ratio of the velocities to them (below 100 here)."""
import numpy as np
import pytest

from oracle import substep as S
from oracle.case import SGS_SMAG, SGS_SMAG_VD
from tests.cases import initial_fields, make_pair, rel_err, say

pytestmark = pytest.mark.gpu
PER, NOSLIP, WM = 0, 1, 2
GRIDS = [(8, 6, 4), (20, 10, 5), (32, 8, 7), (40, 24, 9), (96, 40, 33), (96, 40, 34), (96, 80, 35), (160, 96, 33)]


@pytest.mark.parametrize("zbc,ybc,sgs", [(PER, 0, SGS_SMAG), (NOSLIP, 0, SGS_SMAG), (WM, 0, SGS_SMAG), (WM, 0, SGS_SMAG_VD),
                                         (NOSLIP, 1, SGS_SMAG_VD), (WM, 1, SGS_SMAG), (WM, 1, SGS_SMAG_VD)])
@pytest.mark.parametrize("nx,ny,nz", GRIDS)
def test_strain_at_block_edges(nx, ny, nz, zbc, ybc, sgs):
    from paper_2411_09364_amd import les
    if zbc == PER:
        nz += nz % 2 + (0 if (nz + nz % 2) not in (34, 36) else 40 - (nz + nz % 2))   # a length the transforms take
    case, g, cfg = make_pair(nx, ny, nz, 3.0, 2.0, 2.0, zbc=zbc, ybc=ybc, beta=0.0 if zbc == PER or ybc else 1.2, nu=1e-3,
                             sgs=sgs, cs=0.1)
    u, v, w = initial_fields(case, g, 9, "random")
    st = S.initial_state(case, g, u, v, w)
    solver = les.Solver(cfg)
    solver.set_state(u, v, w)
    solver.nut()
    nut = solver.eddy_viscosity()
    solver.close()
    err = rel_err(nut[:, :ny], st.nut[:, :ny], slice(1, nz + 1))
    say(f"strain {zbc} {nx}x{ny}x{nz} ybc {ybc} sgs {sgs}: {err:.2e}")
    assert np.max(np.abs(st.nut)) > 0 and err < 1e-12
