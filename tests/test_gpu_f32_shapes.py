"""The fp32 products and attention at the edges of their launch shapes,
against the oracle: odd and unaligned feed-forward widths (K % 4 != 0 takes
single loads), both head sizes, vocabulary and row tails, sequences shorter
than one key block, and every product on the large shape (64 x 64 wave tiles)
in one case or another, the head with fewer live rows than its bound; norm
gains on both sides of every fused norm.

Tolerance: logits rel-RMS <= 1e-5 as everywhere on the fp32 path (sums of at
most 2048 products at 2^-24 each, a few roundings deep)."""

import dataclasses

import numpy as np
import pytest
import torch

import paper_2608_01821_amd as dv
import synth
from gpu_util import (TOL, Model, Sample, compare, oracle_step, random_state,
                      run_gpu_step)

pytestmark = pytest.mark.gpu

# d, heads, ffn, vocab, grid, crops, prompt, response, layers, and the products
# that run on the large shape
SHAPES = {
    "short": (64, 1, 33, 17, 2, 1, 1, 3, 2, ""),
    "tails-hd64": (192, 3, 250, 333, 9, 1, 5, 21, 2, ""),
    "unaligned-hd128": (256, 2, 101, 301, 7, 2, 13, 37, 2, ""),
    "large": (768, 12, 520, 9001, 27, 3, 7, 140, 1, "qkv"),
    "large-unaligned": (2048, 16, 65, 1000, 27, 3, 7, 20, 1, "qkv out down"),
    "large-gate-up": (256, 4, 1000, 333, 27, 3, 7, 140, 1, "gate_up"),
    "large-head": (128, 1, 101, 9001, 2, 1, 5, 400, 1, "head"),
}


def large_products(rows, d, ffn, vocab, resp):
    """The launch shape's rule: 128 rows x 4 column pairs (32 columns a pair,
    16 of gate and up) a workgroup once there are 256 of them."""
    products = dict(qkv=(rows, 3 * d, 32), out=(rows, d, 32),
                    gate_up=(rows, ffn, 16), down=(rows, d, 32),
                    head=(resp, vocab, 32))
    return {n for n, (m, cols, pair) in products.items()
            if -(-m // 128) * -(-(-(-cols // pair)) // 4) >= 256}


@pytest.mark.parametrize("name", list(SHAPES))
def test_f32_step_shapes(name):
    d, heads, ffn, vocab, grid, crops, prompt, resp, layers, large = SHAPES[name]
    assert large_products(crops * grid * grid + prompt + resp, d, ffn, vocab,
                          resp) == set(large.split())
    cfg = dataclasses.replace(
        synth.get_any_config(13), n_seqs=1, n_layers=layers, d=d,
        n_heads=heads, head_dim=d // heads, ffn=ffn, vocab=vocab, grid=grid,
        n_crops=crops, prompt_len=prompt, resp_len=resp, crops_range=None,
        prompt_range=None, schedule="fixed", fixed_levels=(2,) * 5)
    rng = np.random.default_rng(len(name))
    mdl = Model(cfg, "f32")
    gains = [rng.uniform(0.5, 1.5, d).astype(np.float32)
             for _ in range(2 * layers + 1)]
    for i in range(layers):
        for j, key in enumerate(("attn_norm", "ffn_norm")):
            mdl.host["layers"][i][key] = gains[2 * i + j]
            mdl.dev_layers[i][key] = torch.from_numpy(gains[2 * i + j]).cuda()
    final = torch.from_numpy(gains[-1]).cuda()
    mdl.host["final_norm"] = gains[-1]
    mdl.weights = dv.Weights(mdl.dev_embed, mdl.dev_head, mdl.dev_layers, final)
    s = synth.gen_sample(cfg)
    sample = Sample(cfg, crops, s["visual"][0], s["prompts"][0], "f32")
    ids, masked = random_state(rng, resp, cfg.mask_id, vocab, 0.7)
    g_conf, g_am, g_lg = run_gpu_step(cfg, mdl, [sample], [2], ids, masked)
    pos, lg, am, cf = oracle_step(cfg, mdl, sample, 2, ids, masked)
    compare(cfg, TOL["f32"], masked, g_conf[0], g_am[0], g_lg[0], pos, lg, am,
            cf)
