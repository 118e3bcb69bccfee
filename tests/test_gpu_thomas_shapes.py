"""The z solves at the edges of their segments and launch shapes: rows that fill a segment of 8 or 16, one row
less and one more, the last count of 64-column and the first of 32-column blocks, the fewest and the most rows;
columns that fill no whole block.  The pressure solve against the oracle's, FP64 and FP32 fields.

Tolerance: that of a backward-stable solve in the stated precision, as for the transforms, |error| <= (10 log2(all
points) + 4 + nz) u |f| / |lambda|: the recurrences of nz rows add one rounding a row (in FP64 for both kinds of
fields, so counted with FP64's u)."""
import numpy as np
import pytest

from oracle import poisson as OP
from tests.cases import make_pair, say

pytestmark = pytest.mark.gpu
NOSLIP = 1


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nz", [4, 7, 8, 9, 16, 17, 32, 33, 95, 96, 97, 104, 105, 127, 128, 129, 192, 193, 208, 256, 511,
                                512])
def test_z_solve_at_segment_edges(nz, precision):
    from paper_2411_09364_amd import les
    for nx, ny, ybc in ((6, 4, 0), (24, 10, 0), (12, 6, 1)):
        case, g, cfg = make_pair(nx, ny, nz, 1.0, 1.0, 1.0, zbc=NOSLIP, ybc=ybc, precision=precision)
        f = np.zeros((nz + 2, getattr(g, "nys", ny), nx))
        f[1:nz + 1, :ny] = np.random.Generator(np.random.PCG64(nz)).standard_normal((nz, ny, nx))
        f[1:nz + 1, :ny] -= f[1:nz + 1, :ny].mean()
        ref = OP.solve(g, f[1:nz + 1])[:, :ny]
        solver = les.Solver(cfg)
        phi = solver.poisson(f)[1:nz + 1, :ny]
        solver.close()
        # the longest wave between walls a unit apart: at least 8
        u = 2.0 ** -24 if precision else 2.0 ** -53
        tol = ((10 * np.log2(nx * ny * nz) + 4) * u + nz * 2.0 ** -53) * np.sqrt(np.sum(f * f)) / 8.0
        err = np.max(np.abs(phi - ref))
        say(f"{nx}x{ny}x{nz} ybc {ybc} precision {precision}: error {err:.2e} of {np.max(np.abs(ref)):.2e}, bound {tol:.1e}")
        assert tol < 0.5 * np.max(np.abs(ref))
        assert err <= tol
