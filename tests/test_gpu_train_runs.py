"""Training sums in a fixed order: a run gives the same bits every time."""
import numpy as np
import pytest

from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,tiles", ((16, 1), (257, 1), (5, 3)))
def test_runs_are_bitwise_equal(blocks, tiles):
    def run():
        g = qed.Generator(capacity=(1, 1, 1))
        cfg = qed.qed_train_config_default()
        cfg.table_chi, cfg.table_x, cfg.steps, cfg.blocks, cfg.batch_tiles = 33, 512, 20, blocks, tiles
        out = qed.qed_train_sampler(g.ctx, cfg)
        g.close()
        return out
    for a, b in zip(run(), run()):
        assert np.array_equal(a, b)
