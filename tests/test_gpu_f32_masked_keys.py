"""fp32 attention where whole 16-key blocks score -inf: a query times a key
overflows fp32 (finite in float64, where its softmax weight is 0), and the
block is some wavefront's first, all of a wavefront's, or nearly all there are.

Rows carry a constant feature 0 and a mark in feature 1.  One query dim reads
the constant, its key dim the mark, both times 1e25, so a marked key scores
-1e50 against every query and an unmarked one 0 from these dims; the dim is
half of the slowest rotary pair (angles below 0.02 at these positions), whose
other half is 0 in queries and keys.

Tolerance: logits rel-RMS <= 1e-5 as everywhere on the fp32 path."""

import dataclasses

import numpy as np
import pytest
import torch

import paper_2608_01821_amd as dv
import synth
from gpu_util import dev_tensor, model_cfg, rel_rms, workspace
from oracle import model

pytestmark = pytest.mark.gpu

# marked view rows (81 of them, then 7 prompt and 12 response rows: 100 keys
# in 7 blocks, taken by wavefronts 0 1 2 3 0 1 2)
MARKED = {
    "none": [],
    "wave-1-first-block": range(16, 32),
    "wave-3-all": range(48, 64),
    "wave-0-all": list(range(16)) + list(range(64, 80)),
    "all-but-two-blocks": range(81),
    "scattered": range(0, 81, 3),
}


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("name", list(MARKED))
def test_blocks_of_minus_infinity(name, head_dim):
    d, L = 2 * head_dim, 12
    cfg = dataclasses.replace(
        synth.get_any_config(13), n_seqs=1, n_layers=1, d=d, n_heads=2,
        head_dim=head_dim, ffn=96, vocab=65, grid=9, n_crops=1, prompt_len=7,
        resp_len=L)
    rng = np.random.default_rng(head_dim)

    def draw(*shape, std=0.05):
        return (std * rng.standard_normal(shape)).astype(np.float32)

    view, embed = draw(81, d, std=1.0), draw(cfg.vocab, d, std=1.0)
    for rows in (view, embed):
        rows[:, 0], rows[:, 1] = 1.0, 0.0
    view[list(MARKED[name]), 1] = 1.0
    layer = dict(wqkv=draw(3 * d, d), wo=draw(d, d), wg=draw(96, d),
                 wu=draw(96, d), wd=draw(d, 96))
    for h in range(2):
        q = h * head_dim + head_dim // 2 - 1
        for row in (q, q + head_dim // 2, d + q, d + q + head_dim // 2):
            layer["wqkv"][row] = 0.0
        layer["wqkv"][q, 0] = 1e25
        layer["wqkv"][d + q, 1] = -1e25
    host = dict(embed=embed, head=draw(cfg.vocab, d), layers=[layer])
    W = dv.Weights(dev_tensor(embed, "f32"), dev_tensor(host["head"], "f32"),
                   [{k: dev_tensor(w, "f32") for k, w in layer.items()}])
    prompt = rng.integers(0, 64, 7).astype(np.int32)
    ids = np.full(L, cfg.mask_id, np.int32)
    masked = np.ones(L, np.uint8)
    conf = torch.empty(L, device="cuda")
    am = torch.empty(L, dtype=torch.int32, device="cuda")
    logits = torch.empty((L, cfg.vocab), device="cuda")
    dv.davet_denoise_step(model_cfg(cfg, "f32"), W, [dev_tensor(view, "f32")],
                          [81], torch.from_numpy(prompt).cuda(), [0, 7],
                          torch.from_numpy(ids).cuda(),
                          torch.from_numpy(masked).cuda(), L, conf, am, logits,
                          workspace(cfg, 100, 1, L, "f32"))
    _, ref = model.step_logits(cfg, view, prompt, ids, masked, host)
    got = logits.cpu().numpy()
    assert np.isfinite(got).all()
    assert rel_rms(got, ref) <= 1e-5
