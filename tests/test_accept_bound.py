"""The acceptance bound of Algorithm 1's kernels bounds eq. (1) wherever it is used.

A test value y at or above c b top_j t_ji / 255 b^(-1/3) (row j: the octave of chi, bin i
of 64 in x) rejects a candidate without F and G; that is the decision of eq. (1) only if
((1 - x^3) F + x^6 G) / x never exceeds the tabulated bound.  The shipped table is evaluated
as the kernels do (float, a few ulps taken off for the hardware's log2 and exp2, the lower
of two rows next to an octave's edge) against the oracle's F and G; the kernels add 0.1%."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INC = os.path.join(ROOT, "paper_2008_10468_amd", "csrc", "accept_coeffs.inc")


def _table():
    src = open(INC).read()
    l0, nrow, nx = (int(re.search(r"#define QED_ACC_%s (-?\d+)" % k, src).group(1)) for k in ("L0", "NROW", "NX"))
    top = np.array([float(v) for v in re.findall(r"([0-9.]+)f", re.search(r"qed_acc_top.*?\};", src, re.S).group(0))],
                   np.float32)
    words = [int(v, 16) for v in re.findall(r"0x([0-9a-f]{8})u", src)]
    t = np.array([(w >> s) & 255 for w in words for s in (0, 8, 16, 24)]).reshape(nrow, nx)
    assert top.size == nrow
    return l0, nrow, nx, top, t


def _bound(chi, l0, nrow, top, t):
    l = np.log2(np.float64(np.float32(chi)))
    rows = {min(max(int(np.floor(l + e)) - l0, 0), nrow - 1) for e in (-1e-5, 1e-5)}
    bm13 = np.exp2(-(np.float32(l) + np.float32(0.58496250072)) * np.float32(1.0 / 3.0))
    return np.min([top[r] * t[r] / 255.0 for r in rows], axis=0) * float(bm13) * (1.0 - 16 * 2.0 ** -24)


@pytest.mark.parametrize("part", range(8))
def test_bound_holds_in_every_cell(orc, part):
    """Every row at 8 chi, every bin at 97 x, the last bin at 400 more towards x = 1; below
    the table's range down to chi = 2^-40, where row 0 serves."""
    l0, nrow, nx, top, t = _table()
    ls = np.concatenate([np.arange(-40, l0) + 0.37, l0 + (np.arange(8 * nrow) + 0.5) / 8.0, l0 + np.arange(nrow + 1)])
    u = (np.arange(97) + 0.5) / 97.0
    x = ((np.arange(nx)[:, None] + u[None, :]) / nx).ravel()
    x = np.concatenate([x, 1.0 - np.logspace(-np.log10(nx), -7.2, 400)])
    i = np.minimum((x * nx).astype(int), nx - 1)
    x3, om = x ** 3, (1.0 - x) * (1.0 + x + x * x)
    for l in ls[part::8]:
        chi = 2.0 ** l
        F, G = orc.synchrotron(np.minimum(x3 / (1.5 * chi * om), 1e3))
        d = (om * F + x3 * x3 * G) / x
        b = _bound(chi, l0, nrow, top, t)[i]
        assert np.all(b >= d * (1.0 + 1e-5)), (l, x[np.argmin(b - d)])


def test_bound_is_close(orc):
    """The squeeze is worth its look-up: the mean over x of the bound stays within 30% of the
    mean of the density (the flat envelope is 1.4 to 10 times it)."""
    l0, nrow, nx, top, t = _table()
    x = (np.arange(64 * 200) + 0.5) / (64 * 200)
    x3, om = x ** 3, (1.0 - x) * (1.0 + x + x * x)
    for l in np.arange(-10, 6) + 0.5:
        F, G = orc.synchrotron(np.minimum(x3 / (1.5 * 2.0 ** l * om), 1e3))
        assert np.mean(_bound(2.0 ** l, l0, nrow, top, t)) <= 1.3 * np.mean((om * F + x3 * x3 * G) / x), l
