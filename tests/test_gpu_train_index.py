"""The indexed bisection of the training table, for row lengths whose bisection ends in
the index, goes past it, and is uneven."""
import numpy as np
import pytest

import oracle
from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", (256, 512, 768, 8192))
def test_samples_invert_the_table(nx):
    """A network of zeros gives y = 0, so the loss of the first step is mean(w y^2) of the
    samples drawn, a function of the table's inversion alone: against a bisection in
    numpy of the same table, with the oracle's random words.  All terms are positive;
    the device rounds each four times and adds at most 290 partial sums in a row, all
    in float: (290 + 4) 2^-24 = 1.8e-5."""
    lo, hi, nchi, seed = -3.0, 2.0, 33, 9
    g = qed.Generator(capacity=(1, 1, 1))
    cdf, _ = qed.qed_emission_cdf(g.ctx, lo, hi, nchi, nx)
    cfg = qed.qed_train_config_default()
    cfg.log10_chi_lo, cfg.log10_chi_hi, cfg.table_chi, cfg.table_x = lo, hi, nchi, nx
    cfg.steps, cfg.seed = 1, seed
    loss = qed.qed_train_sampler(g.ctx, cfg, np.zeros(qed.QED_MLP_NPARAMS, np.float32))[1][0]
    g.close()

    n = cfg.blocks * 64 * cfg.batch_tiles
    ctr = np.zeros((n, 4), np.uint32)
    ctr[:, 0] = np.arange(n)
    key = np.tile(np.array([seed ^ 0x7F4A7C15, 0xF39CC060], np.uint32), (n, 1))
    r = oracle.philox(ctr, key)
    word = lambda p, q: (((p.astype(np.uint64) << np.uint64(32)) | q) >> np.uint64(12)) * np.uint64(2) + np.uint64(1)
    tl, tv = word(r[:, 0], r[:, 1]) * 2.0 ** -53, word(r[:, 2], r[:, 3]) * 2.0 ** -53
    u = -np.expm1(-(2.6 * tv) ** 3)
    l10 = lo + (hi - lo) * tl
    cpos = (l10 - lo) / (hi - lo) * (nchi - 1)
    j = np.clip(np.floor(cpos).astype(int), 0, nchi - 2)
    w = np.clip(cpos - j, 0.0, 1.0)
    m = lambda k: cdf[j, k] + w * (cdf[j + 1, k] - cdf[j, k])
    a, b = np.zeros(n, int), np.full(n, nx)
    while np.any(b - a > 1):
        mid = (a + b) // 2
        right = (m(mid) <= u) & (b - a > 1)
        b = np.where(right | (b - a <= 1), b, mid)
        a = np.where(right, mid, a)
    dm = m(b) - m(a)
    f = np.where(dm > 0.0, (u - m(a)) / np.where(dm > 0.0, dm, 1.0), 0.5)
    xi = (a + f) / nx
    x = 1.0 - (1.0 - xi) ** 2
    chi = 1.5 * 10.0 ** l10
    xs = np.cbrt(chi / (1.0 + chi))
    dy = np.minimum(dm * nx / np.maximum(2.0 * (1.0 - xi), 1e-300) * xs, 5.0)
    ref = np.mean((dy * dy + 1e-4) * (x / xs) ** 2)
    assert abs(loss - ref) <= 1.8e-5 * ref
