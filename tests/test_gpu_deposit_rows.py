"""The deposit's row-wise tile count (many particles and tiles) at the edges of its rows and
of its range, against the oracle."""
import numpy as np
import pytest

from oracle import grid as og
from test_gpu_grid import _deposit_mode, _grid, _particles

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec_name", ["F64", "MIXED"])
@pytest.mark.parametrize("dims", [(57, 49, 61), (128, 128, 64), (129, 128, 64)])   # 3,120, 16,384, 16,896 tiles
@pytest.mark.parametrize("n", (0, 1, 1023, 1025, 262145, 600001))
def test_rows_match_oracle(prec_name, dims, n):
    """One block's row to all 256 of them, partly filled and empty rows; the last grid is one
    tile row beyond the row-wise count, which then leaves it to the other one.  Currents
    agree to 1e-10 of the largest, as for the other deposits (double sums in another order)."""
    from paper_2008_10468_amd import qed
    rng = np.random.default_rng(n + dims[0])
    gen = qed.Generator(precision=getattr(qed, "QED_PREC_" + prec_name), capacity=(1 << 20, 16, 16))
    g, s, _ = _grid(qed, gen.real, rng, *dims)
    p = _particles(g, rng, n)
    if n > 1000:
        p["x"][::97] = np.nan       # off the grid: deposits nothing
        p["ux"][5::89] = np.inf
    gen.sp[0].upload(p)
    _deposit_mode(qed, gen, "sorted")
    q = gen.sp[0].download()
    ok = np.isfinite(q["x"] + q["ux"])
    q = {k: v[ok] for k, v in q.items()}
    ref = og.deposit(g, q["x"], q["y"], q["z"], q["ux"], q["uy"], q["uz"], q["w"], -1.0)
    for _ in range(2):              # the second call meets the first one's scratch
        j = torch.zeros(3, g["nx"] * g["ny"] * g["nz"], dtype=torch.float64, device="cuda")
        assert qed.qed_deposit(gen.ctx, s, gen.sp[0].struct(), -1.0, *[t.data_ptr() for t in j]) == qed.QED_OK
        for t, r in zip(j.cpu().numpy(), ref):
            assert np.abs(t - r).max() <= 1e-10 * max(np.abs(r).max(), 1e-300)
    gen.close()
