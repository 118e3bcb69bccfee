"""Crank-Nicolson in z of columns as tall as the library takes, in FP64 grids whose march has more than eight chunks:
the column solves with the most rows in LDS, in whole-wave blocks (288 rows) and half-wave ones (289 to 512).  A
substep against the oracle within the FP64 substeps' bound of 1e-12 of each component."""
import numpy as np
import pytest

from oracle import substep as S
from oracle.case import SGS_SMAG
from tests.cases import initial_fields, make_pair, rel_err, say

pytestmark = pytest.mark.gpu
NOSLIP, WM = 1, 2


@pytest.mark.parametrize("zbc", [NOSLIP, WM])
@pytest.mark.parametrize("nz", [288, 289, 384, 511, 512])
def test_cn_z_tall_columns(nz, zbc):
    from paper_2411_09364_amd import les
    case, g, cfg = make_pair(10, 8, nz, 3.0, 2.0, 2.0, zbc=zbc, nu=1e-3, sgs=SGS_SMAG, cs=0.1, ubulk=1.0, implicit_z=True)
    u, v, w = initial_fields(case, g, 4, "channel")
    st = S.initial_state(case, g, u, v, w)
    dt = S.time_step(case, g, st, cfl=0.5)
    solver = les.Solver(cfg)
    solver.set_state(u, v, w)
    solver.nut()
    solver.set_dt(dt)
    st = S.substep(case, g, st, 0, dt)
    les.les_timing(solver.ctx, True)
    solver.substep(0)
    les.les_timing(solver.ctx, False)
    got = solver.fields()
    launched = les.les_timing_report(solver.ctx)
    solver.close()
    errs = [rel_err(a, b, slice(1, nz + 1)) for a, b in zip(got, (st.u, st.v, st.w))]
    say(f"cn-z {zbc} 10x8x{nz}: " + " ".join(f"{e:.2e}" for e in errs))
    assert "helmholtz_z" in launched and "hz_factor" not in launched   # not the elimination along the march
    assert max(errs) < 1e-12
