"""The naive scheduler has no limit on the slots of a species: the optical-depth path's queue
of waiting particles holds slots beyond 2^32 as they are."""
import pytest

import workloads
from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _step(n, slots):
    """One step of n electron slots, live at `slots` and with NaN momenta (skipped) elsewhere; to
    fit the card the arrays share memory: x, y, z and the ids (all zero), the momenta and the
    weight.  Per live slot: the optical depth and the last momentum component stored."""
    pos = torch.zeros(n, dtype=torch.float64, device="cuda")
    mom = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    tau = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    mom[list(slots)] = 5.0e3
    g = qed.Generator(precision=qed.QED_PREC_MIXED, capacity=(16, 16, 4096), pairs=False,
                      sampler=qed.QED_SAMPLER_SURROGATE)
    e = g.sp[0]
    e.x = e.y = e.z = e.id = pos
    e.ux = e.uy = e.uz = e.w = mom
    e.tau, e.parent, e.events, e.capacity = tau, None, None, n
    e.n.fill_(n)
    f = workloads.uniform_field(bx=1.0e-3)
    g.fields = [qed.FieldBuffers(f, g.real) for _ in range(3)]
    g.step(2.0e5, 3, 0)
    status, rep = g.sync()
    assert status == qed.QED_ERR_NONFINITE and rep.nonfinite == n - len(slots)
    assert g.stats().substeps[0] > 2 * len(slots)     # more than one sub-step: they are queued
    out = [(float(tau[s]), float(mom[s])) for s in slots]
    g.close()
    return out


def test_slots_beyond_32_bits():
    far = (1 << 32) + 5
    if torch.cuda.get_device_properties(0).total_memory < 120 << 30:
        pytest.skip("needs 86 GB")
    ref = _step(64, (5,))[0]
    assert ref[0] > 0.0 and ref[1] != 5.0e3
    got = _step(far + 59, (5, far))
    torch.cuda.empty_cache()
    assert got == [ref, ref]
