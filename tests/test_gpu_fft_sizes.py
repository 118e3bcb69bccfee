"""Every pass of the LDS transforms, first, middle and last, along x, y (Fourier and cosine) and periodic z: the
pressure solve against the oracle's for lengths that reach each of them, the shortest and the longest among them.

Tolerance: a radix FFT of N points with accurate factors has an error of at most 5 u log2 N of its result in the
2-norm (u the unit roundoff); forward and inverse transforms with the division (or z solve) between them, whose
smallest eigenvalue is |lambda|, then leave |error| <= (10 log2(all points) + 4) u |f| / |lambda|, the 4 for the
rounding of f, of the eigenvalue's quotient and of the result."""
import numpy as np
import pytest

from oracle import poisson as OP
from tests.cases import make_pair, say

pytestmark = pytest.mark.gpu
PER, NOSLIP = 0, 1
LENGTHS = [4, 6, 8, 10, 12, 16, 20, 24, 30, 32, 40, 48, 60, 64, 80, 96, 120, 128, 160, 192, 240, 256, 320, 384, 480, 512,
           640, 768, 960, 1024]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", LENGTHS)
def test_pressure_solve_at_every_length(n, precision):
    from paper_2411_09364_amd import les
    # lengths of 1 in every direction: the smallest eigenvalue is that of the longest wave along z or y walls
    for what, nx, ny, nz, zbc, ybc in (("x", n, 6, 5, NOSLIP, 0), ("y", 12, n, 4, NOSLIP, 0),
                                       ("z", 6, 4, n, PER, 0), ("cosine y", 10, n, 4, NOSLIP, 1)):
        case, g, cfg = make_pair(nx, ny, nz, 1.0, 1.0, 1.0, zbc=zbc, ybc=ybc, precision=precision)
        f = np.zeros((nz + 2, getattr(g, "nys", ny), nx))
        f[1:nz + 1, :ny] = np.random.Generator(np.random.PCG64(n)).standard_normal((nz, ny, nx))
        f[1:nz + 1, :ny] -= f[1:nz + 1, :ny].mean()
        ref = OP.solve(g, f[1:nz + 1])[:, :ny]
        solver = les.Solver(cfg)
        phi = solver.poisson(f)[1:nz + 1, :ny]
        solver.close()
        # second differences of a wave over half a length (walls): at least 8 / length^2
        lam = 8.0
        u = 2.0 ** -24 if precision else 2.0 ** -53
        tol = (10 * np.log2(nx * ny * nz) + 4) * u * np.sqrt(np.sum(f * f)) / lam
        err = np.max(np.abs(phi - ref))
        say(f"{what} {nx}x{ny}x{nz} precision {precision}: error {err:.2e} of {np.max(np.abs(ref)):.2e}, bound {tol:.1e}")
        assert tol < 0.2 * np.max(np.abs(ref))
        assert err <= tol
