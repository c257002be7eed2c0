"""The row-wise tile count of the deposit at tile counts that fill neither its blocks nor its
waves, and at the edges of the rule that chooses it, against the oracle."""
import numpy as np
import pytest

from oracle import grid as og
from paper_2008_10468_amd import qed
from test_gpu_grid import _deposit_mode, _grid, _particles

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# tiles of 4^3 cells: 4,097 = 17 x 241 (one more than the LDS count takes; one tile in the last block of
# 64), 15,625 = 25^3 (9 in the last block of 64), 4,096 and 16,384 (the last of either side), 16,385
@pytest.mark.parametrize("dims", [(65, 961, 1), (99, 98, 97), (64, 64, 64), (128, 128, 64), (20, 452, 113)])
@pytest.mark.parametrize("cap", ((1 << 18), (1 << 18) + 1))   # the capacity's edge: rows from the second on
@pytest.mark.parametrize("prec_name", ["F64", "MIXED"])
def test_edges_match_oracle(prec_name, cap, dims):
    """The buffer full, and one particle in it.  Currents agree to 1e-10 of the largest, as for the
    other deposits (double sums in another order)."""
    tiles = np.prod([(d + 3) // 4 for d in dims])
    assert tiles in (4096, 4097, 15625, 16384, 16385)
    rng = np.random.default_rng(cap + dims[0])
    gen = qed.Generator(precision=getattr(qed, "QED_PREC_" + prec_name), capacity=(cap, 16, 16))
    g, s, _ = _grid(qed, gen.real, rng, *dims)
    _deposit_mode(qed, gen, "sorted")
    for n in (cap, 1):
        p = _particles(g, rng, n)
        if n > 1:
            p["x"][::97] = np.nan       # off the grid: deposits nothing
        gen.sp[0].upload(p)
        q = gen.sp[0].download()
        ok = np.isfinite(q["x"])
        q = {k: v[ok] for k, v in q.items()}
        ref = og.deposit(g, q["x"], q["y"], q["z"], q["ux"], q["uy"], q["uz"], q["w"], -1.0)
        j = torch.zeros(3, g["nx"] * g["ny"] * g["nz"], dtype=torch.float64, device="cuda")
        assert qed.qed_deposit(gen.ctx, s, gen.sp[0].struct(), -1.0, *[t.data_ptr() for t in j]) == qed.QED_OK
        for t, r in zip(j.cpu().numpy(), ref):
            assert np.abs(t - r).max() <= 1e-10 * max(np.abs(r).max(), 1e-300)
    gen.close()
