"""Steps of 16-bit models other than the 8B-shaped one at the edges of what
the planner picks, against the oracle: the phased 256 x 256 tile's rotary QKV
at, one past and between multiples of the tile and of the 64 rows a wave skips,
with one and several bands of row tiles; its gate/up and split down projection;
the same tile as the vocabulary head with a ragged last slab, odd vocabulary
widths and two row tiles; and short sequences whose projections (gate and up
among them) are split over K.  The plans each case is there for are asserted.

Tolerance: logits rel-RMS <= 1e-2 as everywhere on the 16-bit path (one
rounding to 11 or 8 bits of every activation tensor of a layer)."""

import dataclasses

import numpy as np
import pytest
import torch

import paper_2608_01821_amd as dv
import synth
from gpu_util import (DTYPE, TOL, Model, Sample, compare, oracle_step, random_state,
                      run_gpu_step)
from internal import plan_gemm16

pytestmark = pytest.mark.gpu

# d, ffn, mode, vocab, crops (27 x 27), prompt, response, and the (tile, split)
# of QKV, output, gate/up and down
CASES = {
    "whole-tiles": (1024, 1088, "f16", 1024, 4, 84, 72,      # 3072 rows
                    (17, 1), (12, 1), (6, 1), (12, 1)),
    "one-past": (1024, 512, "bf16", 700, 4, 85, 72,          # 3073 rows
                 (17, 1), (12, 1), (12, 1), (12, 1)),
    "row-skip": (1280, 1344, "f16", 700, 4, 120, 100,        # 3136 rows
                 (17, 1), (12, 1), (14, 1), (12, 1)),
    "bands-head": (1024, 512, "f16", 1037, 5, 248, 460,      # 4353 rows
                   (17, 1), (6, 1), (6, 1), (6, 1)),
    "gate-up-down": (2048, 3072, "f16", 700, 3, 18, 100,     # 2305 rows
                     (17, 1), (6, 1), (17, 1), (17, 3)),
    "head-two-tiles": (512, 64, "bf16", 1300, 1, 20, 250,
                       (12, 1), (12, 2), (12, 2), (12, 1)),
    "split-gate-up": (1024, 512, "bf16", 700, 1, 60, 100,    # 889 rows
                      (12, 1), (12, 4), (12, 4), (12, 1)),
    "split-3": (768, 832, "f16", 700, 1, 60, 100,
                (12, 1), (12, 3), (12, 1), (12, 3)),
    "short": (1536, 832, "f16", 700, 0, 7, 60,
              (12, 6), (12, 6), (12, 6), (12, 4)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_planned_products(name):
    d, ffn, mode, vocab, crops, prompt, resp, *plans = CASES[name]
    level = 2 if crops else 0             # 0: its 49 coarsest tokens
    cfg = dataclasses.replace(
        synth.get_any_config(13), n_seqs=1, n_layers=1, d=d, n_heads=d // 128,
        head_dim=128, ffn=ffn, vocab=vocab, grid=27, n_crops=max(1, crops),
        prompt_len=prompt, resp_len=resp, crops_range=None, prompt_range=None,
        schedule="fixed", fixed_levels=(level,) * 5, dtype="bf16")
    rng = np.random.default_rng(len(name))
    mdl = Model(cfg, mode)
    packed = torch.empty(dv.davet_head_tiled_elems(vocab, cfg.d),
                         dtype=mdl.dev_head.dtype, device="cuda")
    dv.davet_pack_head(mdl.dev_head, packed, vocab, cfg.d, DTYPE[mode])
    mdl.weights = dv.Weights(mdl.dev_embed, packed, mdl.dev_layers,
                             head_layout=dv.DAVET_HEAD_TILED)
    s = synth.gen_sample(cfg)
    sample = Sample(cfg, max(1, crops), s["visual"][0], s["prompts"][0], mode)
    rows = sample.sizes[level] + prompt + resp
    for plan, product in zip(plans, ((3 * d, d, True), (d, d, False),
                                     (2 * ffn, d, False), (d, ffn, False))):
        p = plan_gemm16(rows, *product)
        assert (p.tile, p.ksplit) == plan, product
    ids, masked = random_state(rng, resp, cfg.mask_id, vocab,
                               1.0 if "head" in name else 0.7)
    g_conf, g_am, g_lg = run_gpu_step(cfg, mdl, [sample], [level], ids, masked)
    pos, lg, am, cf = oracle_step(cfg, mdl, sample, level, ids, masked)
    compare(cfg, TOL[mode], masked, g_conf[0], g_am[0], g_lg[0], pos, lg, am,
            cf)
