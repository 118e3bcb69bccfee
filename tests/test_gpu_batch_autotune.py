"""The autotuner of a batch times what the batch runs untuned (candidate 0 of chunk lengths and of line groups) and
keeps it unless another candidate is faster."""
import pytest

from oracle.case import SGS_DSM, SGS_SMAG
from tests.cases import initial_fields, make_pair, round32, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,sgs", [(1, SGS_DSM), (0, SGS_DSM), (1, SGS_SMAG)])
def test_untuned_settings_are_candidates(precision, sgs):
    from paper_2411_09364_amd import les
    cases = [make_pair(n, n, n, 3.0, 3.0, 3.0, nu=1e-3, sgs=sgs, cs=0.17, precision=precision) for n in (12, 24, 32, 48)]
    batch = les.Batch([c[2] for c in cases])
    for b, (case, g, cfg) in enumerate(cases):
        batch.set_state(b, *round32(*initial_fields(case, g, b, "random")))
    batch.nut()
    batch.set_dt(1e-4)
    rep = batch.autotune(2)
    say("autotune", precision, sgs, rep)
    batch.close()
    for what in ("kc", "lines"):
        times = rep[what]
        assert set(times) == {"0", "4", "8", "16", "32"}
        assert times[str(rep["chosen"][what])] == min(times.values())
