"""The training kernels at the edges of their blocking."""
import numpy as np
import pytest

from paper_2008_10468_amd import qed

pytestmark = pytest.mark.gpu


def _gradient(params, samples):
    g = qed.Generator(capacity=(1, 1, 1))
    out = qed.qed_mlp_gradient(g.ctx, params, samples)
    g.close()
    return out


@pytest.mark.parametrize("blocks", (1, 2, 255, 256, 257, 512, 513))
def test_gradient_sum_takes_every_block(blocks):
    """Only the samples of the last block, and of block 255 where there is one, carry
    weight: the summed gradient is that of these samples alone, whatever the number of
    blocks.  Both sides round the same products to bfloat16 (relative 2^-8 each), from
    output gradients that differ by the float rounding of 1/n only."""
    rng = np.random.default_rng(blocks)
    params = (rng.standard_normal(qed.QED_MLP_NPARAMS) * 0.15).astype(np.float32)
    n = 64 * blocks
    smp = np.stack([rng.uniform(-1, 1, n), rng.uniform(-1, 1.6, n), rng.uniform(0, 1, n), np.zeros(n)],
                   axis=1).astype(np.float32)
    used = sorted({blocks - 1, min(255, blocks - 1)})
    rows = np.concatenate([np.arange(64 * b, 64 * b + 64) for b in used])
    smp[rows, 3] = 1.0
    loss, grad = _gradient(params, smp)
    loss1, grad1 = _gradient(params, smp[rows])
    share = rows.size / n
    assert abs(loss - loss1 * share) <= 1e-5 * loss1 * share
    assert np.max(np.abs(grad - grad1 * share)) <= 2.0 ** -8 * np.max(np.abs(grad1)) * share


@pytest.mark.parametrize("blocks,tiles", ((16, 1), (8, 2), (5, 3), (1, 16)))
def test_step_does_not_depend_on_the_split(blocks, tiles):
    """One optimizer step over the same samples (they are drawn by their number) in
    another split over blocks and tiles: the loss agrees to the rounding of float sums
    of 1,024 positive terms (1,024 2^-24 = 6e-5).  Adam's first step moves a parameter by
    lr g / (|g| + 1e-8), so parameters move alike but for those whose gradient is
    lost in that rounding or near 1e-8: one in a hundred is allowed."""
    def step(blocks, tiles):
        g = qed.Generator(capacity=(1, 1, 1))
        cfg = qed.qed_train_config_default()
        cfg.table_chi, cfg.table_x, cfg.steps, cfg.blocks, cfg.batch_tiles = 33, 512, 1, blocks, tiles
        params, loss, _, _ = qed.qed_train_sampler(g.ctx, cfg)
        g.close()
        return params, loss[0], cfg.lr
    params, loss, lr = step(blocks, tiles)
    ref, ref_loss, _ = step(blocks * tiles, 1)
    assert abs(loss - ref_loss) <= 6e-5 * ref_loss
    assert np.mean(np.abs(params - ref) > 1e-3 * lr) <= 0.01
