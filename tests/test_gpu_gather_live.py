"""The gather's forms go by the live particles, not by the capacity: at the edges of both rules
a particle's fields are the same bits, and the oracle's values."""
import numpy as np
import pytest

from oracle import grid as og
from paper_2008_10468_amd import qed
from test_gpu_gather_rows import _gather
from test_gpu_grid import COMP, _grid, _particles

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LINES = (1 << 16, 1 << 19)   # corners in any order below the first, in cell order below the second


@pytest.mark.parametrize("nx", (1, 2, 17))
@pytest.mark.parametrize("prec_name", ["F64", "MIXED"])
@pytest.mark.parametrize("line", LINES)
@pytest.mark.parametrize("in_rows", (False, True))
def test_live_counts_around_a_line(line, in_rows, prec_name, nx):
    """One particle fewer than the line, the line and one more, in a buffer with room for twice
    as many.  Tolerance against the oracle as in the other gather tests."""
    rng = np.random.default_rng(line + nx)
    cap = 2 * line
    gen = qed.Generator(precision=getattr(qed, "QED_PREC_" + prec_name), capacity=(cap, 16, 16))
    g, s, _ = _grid(qed, gen.real, rng, nx=nx)
    p = _particles(g, rng, line + 1)
    if in_rows:
        cell = [np.floor((p[k] - g[k + "0"]) / g["d" + k]) % g["n" + k] for k in "xyz"]
        order = np.lexsort(cell)
        p = {k: v[order] for k, v in p.items()}
    p["x"][::1000] = np.inf                       # lanes off the grid inside a wave
    got = [_gather(gen, s, {k: v[:n] for k, v in p.items()}, cap)[:, :n] for n in (line + 1, line, line - 1)]
    gen.close()
    for b in got[1:]:
        assert np.array_equal(got[0][:, :b.shape[1]], b, equal_nan=True)
    on = np.isfinite(p["x"])
    assert np.all(np.isnan(got[0][:, ~on]))
    some = np.flatnonzero(on)[::17]
    ref = og.gather(g, p["x"][some], p["y"][some], p["z"][some])
    tol = 1e-12 if prec_name == "F64" else 2e-6
    for c, v in zip(COMP, got[0][:, some]):
        assert np.abs(v - ref[c]).max() / np.abs(g[c]).max() < tol, c
