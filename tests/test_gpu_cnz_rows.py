"""Crank-Nicolson in z with FP32 fields at the edges of the elimination's row groups: rows held in registers (32
in batches of 16), one more and one less, rows in LDS, the last count of whole-wave blocks (288 rows) and beyond.
A substep against the oracle with the tolerance that the float32 path's substeps have (1e-5 of each component)."""
import numpy as np
import pytest

from oracle import substep as S
from oracle.case import SGS_SMAG
from tests.cases import initial_fields, make_pair, rel_err, round32, say

pytestmark = pytest.mark.gpu
NOSLIP, WM = 1, 2


@pytest.mark.parametrize("zbc,ybc", [(NOSLIP, 0), (WM, 0), (WM, 1)])
@pytest.mark.parametrize("nz", [4, 15, 16, 17, 31, 32, 33, 34, 47, 48, 49, 50, 75, 287, 288, 289, 290])
def test_cn_z_rows(nz, zbc, ybc):
    from paper_2411_09364_amd import les
    nx, ny = (10, 8) if nz > 100 else (24, 10)     # columns that fill no whole wave
    case, g, cfg = make_pair(nx, ny, nz, 3.0, 2.0, 2.0, zbc=zbc, ybc=ybc, nu=1e-3, sgs=SGS_SMAG, cs=0.1, ubulk=1.0,
                             implicit_z=True, precision=1)
    u, v, w = round32(*initial_fields(case, g, 4, "duct" if ybc else "channel"))
    st = S.initial_state(case, g, u, v, w)
    dt = S.time_step(case, g, st, cfl=0.5)
    solver = les.Solver(cfg)
    solver.set_state(u, v, w)
    solver.nut()
    solver.set_dt(dt)
    st = S.substep(case, g, st, 0, dt)
    solver.substep(0)
    got = solver.fields()
    solver.close()
    I = slice(1, nz + 1)
    errs = [rel_err(a[:, :ny], b[:, :ny], I) for a, b in zip(got, (st.u, st.v, st.w))]
    say(f"cn-z {zbc} {nx}x{ny}x{nz} ybc {ybc}: " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) < 1e-5
