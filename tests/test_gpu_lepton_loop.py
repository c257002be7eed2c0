"""Algorithm 1's loop at the edges of its waiting lanes and of the block's photon pool:
particle by particle against the oracle."""
import pytest

import workloads
from gpu_util import check_step
from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 63, 64, 65, 256, 1500))
@pytest.mark.parametrize("batch", (1, 16, 64))
def test_ring_electrons_match_oracle(n, batch):
    """FP64 electrons in a ring field eight times as strong over four times the step: several
    emissions each, so that at 1,500 electrons blocks fill their pool (224 photons a half)
    many times over, and odd counts leave partly filled waves.  The double path takes every
    decision as the oracle does: all events identical, momenta to 1e-9 as in the other
    FP64 comparisons."""
    w = workloads.c1(n=n, seed=100 + n)
    f = workloads.uniform_field(bz=8.0 * workloads.B_C1)
    g = qed.Generator(precision=qed.QED_PREC_F64, capacity=(n, 16, 64 * n + 4096), pairs=False)
    t = qed.qed_get_tuning(g.ctx)
    t.resolve_batch = batch
    assert qed.qed_set_tuning(g.ctx, t) == qed.QED_OK
    g.load_state(w)
    g.set_fields(f)
    out, after, _ = check_step(g, f, 4.0 * w["dt"], 7, 3, qed.QED_PREC_F64, pairs=False, rtol=1e-9)
    assert out["electron"] == 1.0
    assert n < 64 or after[2]["id"].size > 2 * n
    g.close()
