"""The transforms' passes that only odd lengths reach, along a periodic z (5 points: one stage and the copy pass; 15:
radix 5, then a last pass of radix 3 alone): the pressure solve, and Crank-Nicolson in all directions with its
three components at once, against the oracle; tolerances as in test_gpu_fft_sizes.py and of the FP64 substeps."""
import numpy as np
import pytest

from oracle import poisson as OP
from oracle import substep as S
from oracle.case import SGS_SMAG
from tests.cases import initial_fields, make_pair, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny,nz", [(6, 4, 5), (24, 10, 5), (6, 4, 15), (40, 12, 15)])
def test_pressure_solve_of_odd_plane_counts(nx, ny, nz, precision):
    from paper_2411_09364_amd import les
    case, g, cfg = make_pair(nx, ny, nz, 1.0, 1.0, 1.0, precision=precision)
    f = np.zeros((nz + 2, ny, nx))
    f[1:nz + 1] = np.random.Generator(np.random.PCG64(nz)).standard_normal((nz, ny, nx))
    f[1:nz + 1] -= f[1:nz + 1].mean()
    ref = OP.solve(g, f[1:nz + 1])
    solver = les.Solver(cfg)
    phi = solver.poisson(f)[1:nz + 1]
    solver.close()
    # the longest wave of four points and more over a unit length: 4 / h^2 sin^2(pi / n) >= 32
    u = 2.0 ** -24 if precision else 2.0 ** -53
    tol = (10 * np.log2(nx * ny * nz) + 4) * u * np.sqrt(np.sum(f * f)) / 32.0
    err = np.max(np.abs(phi - ref))
    say(f"{nx}x{ny}x{nz} precision {precision}: error {err:.2e} of {np.max(np.abs(ref)):.2e}, bound {tol:.1e}")
    assert tol < 0.2 * np.max(np.abs(ref))
    assert err <= tol


@pytest.mark.parametrize("nz", [5, 15])
def test_cn_in_all_directions_with_odd_plane_counts(nz):
    from paper_2411_09364_amd import les
    case, g, cfg = make_pair(16, 12, nz, 3.0, 2.0, 2.0, nu=1e-2, sgs=SGS_SMAG, cs=0.1, implicit_3d=True)
    u, v, w = initial_fields(case, g, 5, "random")
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
    errs = [rel_err(a, b, slice(1, nz + 1)) for a, b in zip(got, (st.u, st.v, st.w))]
    say(f"cn-3d periodic 16x12x{nz}: " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) < 1e-12
