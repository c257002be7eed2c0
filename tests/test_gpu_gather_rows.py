"""The gather's forms, chosen by the capacity and by how often a wave's lanes change their row
of cells: the same bits in any of them and in any order, and the oracle's values."""
import numpy as np
import pytest

from oracle import grid as og
from paper_2008_10468_amd import qed
from test_gpu_grid import COMP, _grid, _particles

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gather(gen, s, p, n):
    gen.sp[0].upload(p)
    out = [torch.full((n,), float("nan"), dtype=gen.real, device="cuda") for _ in COMP]
    assert qed.qed_gather(gen.ctx, s, gen.sp[0].struct(), [t.data_ptr() for t in out]) == qed.QED_OK
    torch.cuda.synchronize()
    return np.stack([t.double().cpu().numpy() for t in out])


# one below, at and above the capacity from which pairs are read; rows of one point (no
# pairs), two (every pair ends a row), an odd number
@pytest.mark.parametrize("n", (65535, 65536, 65600))
@pytest.mark.parametrize("nx", (1, 2, 17))
@pytest.mark.parametrize("prec_name", ["F64", "MIXED"])
def test_any_order_gives_the_same_bits(n, nx, prec_name):
    """Positions in random order, and the same sorted by cell row: every particle's fields
    agree bit for bit.  Against the oracle as in the other gather tests."""
    rng = np.random.default_rng(n + nx)
    gen = qed.Generator(precision=getattr(qed, "QED_PREC_" + prec_name), capacity=(n, 16, 16))
    g, s, dev = _grid(qed, gen.real, rng, nx=nx)
    p = _particles(g, rng, n)
    p["x"][::1000] = np.inf                       # lanes off the grid inside a wave
    a = _gather(gen, s, p, n)
    cell = [np.floor((np.where(np.isfinite(p[k]), p[k], 0.0) - g[k + "0"]) / g["d" + k]) % g["n" + k] for k in "xyz"]
    order = np.lexsort(cell)
    b = _gather(gen, s, {k: v[order] for k, v in p.items()}, n)
    gen.close()
    gen = qed.Generator(precision=getattr(qed, "QED_PREC_" + prec_name), capacity=(2 * n, 16, 16))
    assert np.array_equal(_gather(gen, s, p, 2 * n)[:, :n], a, equal_nan=True)   # above the line for every n
    gen.close()
    assert np.array_equal(a[:, order], b, equal_nan=True)
    on = np.isfinite(p["x"])
    assert np.all(np.isnan(a[:, ~on]))
    ref = og.gather(g, p["x"][on], p["y"][on], p["z"][on])
    tol = 1e-12 if prec_name == "F64" else 2e-6
    for c, got in zip(COMP, a[:, on]):
        assert np.abs(got - ref[c]).max() / np.abs(g[c]).max() < tol, c
