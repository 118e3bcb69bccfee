"""Predictor chunks of every length and the Helmholtz factors formed beside it: grids whose launches make no whole
rounds, from one plane a chunk to chunks that end within the last one, in FP64 and FP32 fields, explicit and
implicit; a substep against the oracle, within 1e-11 and 1e-5 of the largest velocity (the bounds of the substeps'
own tests, there of each component)."""
import numpy as np
import pytest

from oracle import substep as S
from oracle.case import SGS_SMAG
from tests.cases import initial_fields, make_pair, round32, say

pytestmark = pytest.mark.gpu
PER, NOSLIP, WM = 0, 1, 2


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("visc", ["explicit", "cn-z", "cn-3d"])
@pytest.mark.parametrize("zbc,nx,ny,nz", [(PER, 16, 12, 4), (PER, 32, 32, 32), (NOSLIP, 12, 6, 4), (NOSLIP, 24, 20, 9),
                                          (WM, 24, 10, 17), (WM, 40, 24, 65), (NOSLIP, 120, 96, 75), (WM, 96, 120, 67)])
def test_predictor_chunk_lengths(zbc, nx, ny, nz, visc, precision):
    from paper_2411_09364_amd import les
    if zbc == PER and visc == "cn-z":
        pytest.skip("CN in z takes walls")
    case, g, cfg = make_pair(nx, ny, nz, 3.0, 2.0, 2.0, zbc=zbc, nu=1e-3, sgs=SGS_SMAG, cs=0.1,
                             ubulk=0.0 if zbc == PER else 1.0, implicit_z=visc == "cn-z", implicit_3d=visc == "cn-3d",
                             precision=precision)
    u, v, w = initial_fields(case, g, 6, "random" if zbc == PER else "channel")
    if precision:
        u, v, w = round32(u, v, w)
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
    ref = (st.u, st.v, st.w)
    top = max(np.max(np.abs(b[I])) for b in ref)
    errs = [np.max(np.abs(a[I] - b[I])) / top for a, b in zip(got, ref)]
    say(f"predictor {zbc} {nx}x{ny}x{nz} {visc} precision {precision}: " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) < (1e-5 if precision else 1e-11)
