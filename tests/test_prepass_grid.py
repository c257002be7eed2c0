"""The pre-pass's default grid is what the chip holds at once (kPrepassBlocks blocks per compute
unit, on which the compiled registers and LDS of k_prepass<float> rest), and a grid that the
caller sets is kept."""
import os
import re

import pytest

from test_kernel_resources import ROOT, _one, usage  # noqa: F401  (usage: the compiler's report)


def _resident():
    src = open(os.path.join(ROOT, "paper_2008_10468_amd", "csrc", "qed_internal.hpp")).read()
    return [int(v) for v in re.search(r"kPrepassBlocks\[2\] = \{(\d+), (\d+)\}", src).groups()]


def test_resident_blocks(usage):  # noqa: F811
    """A block of 256 threads is one wave on each of a compute unit's four SIMDs."""
    for blocks, args in zip(_resident(), ("IfLb0E", "IfLb1E")):
        f = _one(usage, "k_prepass", args)
        assert f["occ"] >= blocks and blocks * f["lds"] <= 160 * 1024 and f["scratch"] == 0


@pytest.mark.gpu
def test_default_grid():
    from paper_2008_10468_amd import qed
    for blocks, sampler in zip(_resident(), (qed.QED_SAMPLER_REJECTION, qed.QED_SAMPLER_SURROGATE)):
        g = qed.Generator(capacity=(16, 16, 16), sampler=sampler)
        t = qed.qed_get_tuning(g.ctx)
        assert t.prepass_blocks_per_cu == blocks
        g.close()
