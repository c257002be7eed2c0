"""Offline generator of the acceptance bound of Algorithm 1 (writes
``csrc/accept_coeffs.inc``).

A candidate x of Algorithm 1 is accepted if its test value y is below
3 x^2 P(x^3) = c b D(x), D(x) = ((1 - x^3) F(z) + x^6 G(z)) / x, z = x^3 / (b (1 - x^3)).
With x in one of NX equal bins (the top bits of its random word) and chi in one
octave, D b^(1/3) is at most top_j t_ji / 255: the table holds top_j as a float and
t_ji as a byte, rounded up, 1% above the largest value found in the cell (9 chi times 24
x per cell, the octave widened by 0.1% on both sides, the last cell refined towards x = 1).  A y above the bound rejects
without F and G, and a y below it is accepted in about nine cases of ten.

Below 2^L0 the first row holds too: there D b^(1/3) depends on z alone, and at a given
x a smaller b means a larger z, a smaller value.
Run: ``python -m paper_2008_10468_amd.fitgen.accept_bound``.
"""
from __future__ import annotations

import os
import sys

import numpy as np

from . import rate_fit

L0 = -16          # chi = 2^-16 ...
NROW = 28         # ... to 2^12, one row per octave
NX = 64
MARGIN = 1.01


def density(x, b, grid):
    t, z, F, G = grid
    d = (1.0 - x) * (1.0 + x + x * x)
    zz = x ** 3 / (b * d)
    lz = np.log(zz)
    inside = (lz > t[0]) & (lz < t[-1])
    Fi = np.where(inside, np.exp(np.interp(lz, t, np.log(np.maximum(F, 1e-300)))), 0.0)
    Gi = np.where(inside, np.exp(np.interp(lz, t, np.log(np.maximum(G, 1e-300)))), 0.0)
    small = lz <= t[0]       # series limit F ~ 2.1495 z^(1/3), G ~ 1.0748 z^(1/3)
    Fi = np.where(small, 2.1495282415344787 * zz ** (1.0 / 3.0), Fi)
    Gi = np.where(small, 1.0747641207672394 * zz ** (1.0 / 3.0), Gi)
    return (d * Fi + x ** 6 * Gi) / x


def table(grid):
    """top[j] and t[j][i]."""
    x = (np.arange(NX)[:, None] + np.linspace(0.0, 1.0, 24)[None, :]) / NX
    x = np.clip(x, 1e-9, 1.0 - 1e-9)
    edge = 1.0 - np.logspace(-np.log10(NX), -9.0, 600)   # the spectrum of large chi: 1 - x ~ 1 / b
    top, cells = [], []
    for j in range(NROW):
        m = np.zeros(NX)
        for l in L0 + j + np.linspace(-0.001, 1.001, 9):
            b = 1.5 * 2.0 ** l
            d = density(x, b, grid).max(axis=1)
            d[-1] = max(d[-1], density(edge, b, grid).max())
            m = np.maximum(m, d * b ** (1.0 / 3.0))
        m *= MARGIN
        top.append(np.float32(m.max() * (1.0 + 1e-6)))
        cells.append(np.ceil(255.0 * m / float(top[-1])).astype(int))
    return top, cells


def main(out_path=None):
    here = os.path.dirname(os.path.abspath(__file__))
    out_path = out_path or os.path.join(os.path.dirname(here), "csrc", "accept_coeffs.inc")
    top, cells = table(rate_fit._fg_grid())
    assert max(max(c) for c in cells) <= 255
    lines = [
        "// Generated by paper_2008_10468_amd/fitgen/accept_bound.py -- do not edit.",
        "// ((1 - x^3) F(z) + x^6 G(z)) / x <= top[j] t[j][i] / 255 b^(-1/3) for x in bin i of",
        f"// {NX} and chi in [2^(QED_ACC_L0 + j), 2^(QED_ACC_L0 + j + 1)]; row 0 also below.",
        f"#define QED_ACC_L0 {L0}",
        f"#define QED_ACC_NROW {NROW}",
        f"#define QED_ACC_NX {NX}",
        f"QED_ACC_STORAGE float qed_acc_top[{NROW}] = {{",
    ]
    for j in range(0, NROW, 7):
        lines.append("  " + ", ".join(repr(float(v)) + "f" for v in top[j:j + 7]) + ",")
    lines += ["};", "// four bins per word, the lowest in the low byte",
              f"QED_ACC_STORAGE unsigned int qed_acc_t[{NROW}][{NX // 4}] = {{"]
    for c in cells:
        words = [c[i] | c[i + 1] << 8 | c[i + 2] << 16 | c[i + 3] << 24 for i in range(0, NX, 4)]
        lines.append("  {" + ", ".join("0x%08xu" % w for w in words) + "},")
    lines.append("};")
    with open(out_path, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("wrote", out_path, file=sys.stderr)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else None)
