"""Algorithm 1's float loop (two sub-steps per Philox block, the second made up after a wait): its
results do not depend on how many lanes wait before they are resolved."""
import numpy as np
import pytest

import workloads
from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu

FIELDS = {"magnetic": dict(bz=4.0e-3), "electric": dict(ex=3.0e-3, ey=-2.0e-3),
          "general": dict(ex=2.0e-3, ez=1.0e-3, by=3.0e-3, bz=-2.0e-3)}


def _run(n, field, sched, batch, dt):
    g = qed.Generator(precision=qed.QED_PREC_MIXED, capacity=(n, 16, 64 * n + 4096), pairs=False,
                      scheduler=getattr(qed, "QED_SCHED_" + sched))
    t = qed.qed_get_tuning(g.ctx)
    t.resolve_batch = batch
    t.light_max = 6          # binned: both the light pass and the heavy queue take particles
    assert qed.qed_set_tuning(g.ctx, t) == qed.QED_OK
    g.load_state(workloads.c1(n=n, seed=40 + n))
    g.set_fields(workloads.uniform_field(**FIELDS[field]))
    for step in range(2):
        g.step(dt, 7, step)
        assert g.sync()[0] == qed.QED_OK
    s = g.stats()
    e, ph = g.sp[0].download(), g.sp[2].download()
    ev = g.sp[0].events_host(n)
    g.close()
    order = np.argsort(ph["id"])
    return e, {k: v[order] for k, v in ph.items()}, ev, (s.substeps[0], s.emissions, s.clips, s.max_p)


@pytest.mark.parametrize("sched", ("NAIVE", "TILED", "BINNED"))
@pytest.mark.parametrize("field", sorted(FIELDS))
@pytest.mark.parametrize("n", (1, 65, 1500))
def test_results_do_not_depend_on_the_batch(n, field, sched):
    """Batches of 1, 16 and 64: electrons, events, photons by id and the counters bit for bit.  The
    population's sub-step counts are odd and even, with several emissions a particle."""
    dt = 2.0 * workloads.c1(n=1)["dt"]
    ref = _run(n, field, sched, 16, dt)
    assert n < 65 or ref[3][1] > n // 4
    for batch in (1, 64):
        got = _run(n, field, sched, batch, dt)
        for a, b in zip(ref[:2], got[:2]):
            assert a.keys() == b.keys()
            for k in a:
                assert np.array_equal(a[k], b[k]), (batch, k)
        assert np.array_equal(ref[2], got[2]) and ref[3] == got[3], batch
