"""The tiles of the light pass and of the tile-sorted scheduler follow the number of
particles: at the counts where the size changes every particle is taken once, with
the bits of the unsorted scheduler."""
import numpy as np
import pytest

import workloads
from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu


def _step(n, sched, tuning):
    w = workloads.c2(n_e=n, n_g=16, seed=5)
    g = qed.Generator(precision=qed.QED_PREC_MIXED, capacity=(n + 4096, 4096, 1 << 18), scheduler=sched)
    t = qed.qed_get_tuning(g.ctx)
    for k, v in tuning.items():
        setattr(t, k, v)
    assert qed.qed_set_tuning(g.ctx, t) == qed.QED_OK
    g.load_state(w)
    g.set_fields(workloads.c2_field(0))
    g.step(w["dt"], 5, 0)
    assert g.sync()[0] == qed.QED_OK
    out = [g.sp[k].download() for k in (0, 2)]
    sub = list(g.stats().substeps)
    g.close()
    return [{k: d[k][np.argsort(d["id"])] for k in ("id", "ux", "uy", "uz", "x", "y", "z")} for d in out], sub


# 2,048 waves on the 256 CUs: 64 slots each up to 131,072 particles, then 128, 192, ...
@pytest.mark.parametrize("n", (1, 65, 131072, 131073, 393217, 1048577))
def test_tiles_match_unsorted(n):
    ref, sub = _step(n, qed.QED_SCHED_NAIVE, {})
    for sched, tuning in ((qed.QED_SCHED_TILED, {}), (qed.QED_SCHED_TILED, {"tiled_slots": 64}),
                          (qed.QED_SCHED_BINNED, {"light_max": 8, "prepass_finish": 0})):
        got, sub2 = _step(n, sched, tuning)
        assert sub == sub2
        for a, b in zip(ref, got):
            for k in a:
                assert np.array_equal(a[k], b[k]), (sched, tuning, k)
