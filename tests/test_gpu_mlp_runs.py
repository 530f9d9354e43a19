"""The loss gradient where a wavefront takes runs of four tiles (from 8192 tiles
of 32 samples on), the last run whole or partial, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


# 8191 tiles (single ones), 8192 with one sample in the last, 8192 full, one more (a run of one), an odd rest
@pytest.mark.parametrize("n", [262112, 262113, 262144, 262145, 300007])
@pytest.mark.parametrize("tau", [0.0, 0.2])
def test_gradient_runs(n, tau):
    import paper_2010_03567_amd.g4hip as g
    ctx = g.Context()
    rng = np.random.default_rng(n)
    w = rng.normal(size=oracle.NPARAM)
    w[:512] /= 8 ** 0.5
    w[576:4672] /= 8
    w[4736:4800] /= 8
    w = torch.from_numpy(w.astype(np.float32)).to(torch.bfloat16)
    feat = rng.normal(size=(n, 8)).astype(np.float32)
    tgt = (rng.normal(size=n) - 1.0).astype(np.float32)  # y - target has a mean, so every run counts in dL/db3
    grad, loss = g.g4_mlp_grad(ctx, w.cuda(), torch.from_numpy(feat).cuda(), torch.from_numpy(tgt).cuda(), tau)
    lref, gref = oracle.mlp_loss_grad(w.double().numpy(), feat.astype(np.float64), tgt.astype(np.float64), tau)
    assert loss.item() == pytest.approx(lref, rel=1e-5)
    gg = grad.cpu().numpy()
    # FP32 terms of both signs, 1e-6 of the sum of their magnitudes; the pinball loss changes slope where
    # FP32 and FP64 disagree on the sign of y - target: 1 / n each, for a few samples
    flips = 4.0 / n if tau > 0 else 0.0
    for sl in (slice(0, 512), slice(512, 576), slice(576, 4672), slice(4672, 4736), slice(4736, 4800)):
        assert np.abs(gg[sl] - gref[sl]).max() <= 2e-5 * np.abs(gref).max() + flips, sl
    # dL/db3 adds the sums of n / 128 runs one after the other, each rounded to 2^-24 of the total at worst
    # (a quarter of the mean run, where the mean is not small against the samples' spread)
    b3 = gref[4800]
    assert abs(gg[4800] - b3) <= (n / 128) * 2.0 ** -24 * abs(b3) + flips + 2e-6 * np.abs(gref).max()
