"""Static model in batches: a batch's |S| kernel against the single context's, in FP32 and FP64, on boxes narrower
than a tile, with remainders and with an odd plane count: every bit of nu_t and of the fields after a step."""
import numpy as np
import pytest

from oracle.case import SGS_SMAG
from tests.cases import initial_fields, make_pair, round32, say

pytestmark = pytest.mark.gpu
BOXES = [(8, 6, 4), (20, 12, 5), (32, 8, 15), (40, 24, 16), (96, 40, 30), (64, 64, 64)]


@pytest.mark.parametrize("precision", [0, 1])
def test_static_batch_equals_single_contexts(precision):
    from paper_2411_09364_amd import les
    cases = [make_pair(nx, ny, nz, 3.0, 2.0, 2.0, nu=1e-3, sgs=SGS_SMAG, cs=0.17, precision=precision)
             for nx, ny, nz in BOXES]
    batch = les.Batch([c[2] for c in cases])
    singles = []
    for b, (case, g, cfg) in enumerate(cases):
        f = round32(*initial_fields(case, g, 30 + b, "random"))
        batch.set_state(b, *f)
        s = les.Solver(cfg)
        s.set_state(*f)
        s.nut()
        singles.append(s)
    batch.nut()
    for b, s in enumerate(singles):
        assert np.array_equal(batch.eddy_viscosity(b), s.eddy_viscosity()), BOXES[b]
    batch.set_dt(1e-3)
    for s in singles:
        s.set_dt(1e-3)
    for k in range(3):
        batch.substep(k)
        for s in singles:
            s.substep(k)
    for b, s in enumerate(singles):
        nut = batch.eddy_viscosity(b)
        say(f"static batch precision {precision} box {BOXES[b]}: largest nu_t {np.max(nut):.2e}")
        assert np.max(nut) > 0 and np.array_equal(nut, s.eddy_viscosity()), BOXES[b]
        for q, (x, y) in enumerate(zip(batch.fields(b), s.fields())):
            assert np.array_equal(x, y), (BOXES[b], q)
        s.close()
    batch.close()
