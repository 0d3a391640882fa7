"""The RMSNorm fused into the fp32 products, at the largest width: rows of
equal magnitude, where additions in one long chain round the same way each
time and a sum of 8192 squares can lose 1e-5.

A model of no layers and a head of unit vectors: logit k of a masked row is
element k of the normed [MASK] embedding, without sums of its own.  In both
launch shapes (the head's 128-row tiles start at 256 workgroups).

Tolerance 8 * 2^-24 relative: two roundings of the squares and of their sums
of four, a few of the compensated sum and the lanes' additions, halved by the
square root; the mean, root, quotient and product one each.  Squares that overflow make the norm's
factor 0, not NaN."""

import numpy as np
import pytest
import torch

import paper_2608_01821_amd as dv

pytestmark = pytest.mark.gpu
D = 8192


@pytest.mark.parametrize("rows,vocab", [(3, 70), (1000, 4100)])
def test_sum_of_equal_squares(rows, vocab):
    assert (-(-rows // 128) * -(-vocab // 128) >= 256) == (rows > 3)
    cfg = dv.ModelCfg(0, D, D // 128, 128, 64, vocab, vocab - 1, 1e-5, 1e4,
                      dv.DAVET_F32)
    rng = np.random.default_rng(vocab)
    embed = torch.zeros((vocab, D), device="cuda")
    W = dv.Weights(embed, torch.eye(vocab, D, device="cuda"), [])
    masked = torch.zeros(rows, dtype=torch.uint8, device="cuda")
    masked[[0, rows // 2, rows - 1]] = 1
    ids = torch.zeros(rows, dtype=torch.int32, device="cuda")
    conf = torch.empty(rows, device="cuda")
    am = torch.empty(rows, dtype=torch.int32, device="cuda")
    logits = torch.empty((rows, vocab), device="cuda")
    prompt = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(dv.davet_workspace_bytes(cfg, rows + 1, 1, rows),
                     dtype=torch.uint8, device="cuda")
    for c in np.append(np.exp(rng.uniform(-3, 3, 12)), 1e20).astype(np.float32):
        x = c * np.where(rng.random(D) < 0.5, -1, 1).astype(np.float32)
        embed[vocab - 1] = torch.from_numpy(x)
        dv.davet_denoise_step(cfg, W, [None], [0], prompt, [0, 1], ids, masked,
                              rows, conf, am, logits, ws)
        if c > 1e19:
            assert (logits[masked.bool()] == 0).all()
            continue
        x = x.astype(np.float64)
        ref = x / np.sqrt(np.mean(x * x) + np.float64(np.float32(1e-5)))
        got = logits[masked.bool()].cpu().numpy()
        assert np.max(np.abs(got / ref[:vocab] - 1)) <= 8 * 2.0 ** -24
