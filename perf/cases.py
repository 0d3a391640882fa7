"""Performance cases of the DAVET hot path on one MI355X.

Each case is one call (or the few calls a program makes together) through the
package's public entry points:

  views   davet_build_views: the evidence hierarchy of one sample
  commit  davet_unmask + davet_policy_step_device: what ends a step
  loop    davet_run_schedule: the whole loop of the small fp32 model under the
          allocation policy (views, T steps, commitments, policy steps)
  step    davet_denoise_step: one step of a 16-bit model

The 16-bit cases are single steps: a whole 16-bit loop turns a last-bit
difference of one confidence into another commitment and from there into
another sequence, so its later outputs say nothing about precision.  A step
returns the logits of its masked rows and their confidences.  Its argmaxes are
not returned: they are the argmaxes of the returned logits, and near-tied ones
change with any change of rounding.
"""

import math
import random

import numpy as np
import torch

import paper_2608_01821_amd as dv

DTYPES = {"f32": (torch.float32, dv.DAVET_F32),
          "bf16": (torch.bfloat16, dv.DAVET_BF16),
          "f16": (torch.float16, dv.DAVET_F16)}
REALIZERS = {"pool": dv.DAVET_REALIZER_POOL, "mixed": dv.DAVET_REALIZER_POOL,
             "prune": dv.DAVET_REALIZER_PRUNE, "merge": dv.DAVET_REALIZER_MERGE}
THETA, EPS = 10000.0, 1e-5


# ------------------------------------------------------------------- cases --

def _views(name, **kw):
    c = dict(kind="views", realizer="pool", dtype="f16", crops=1, grid=27,
             d=4096, K=3, stride=0)
    c.update(kw, name=name)
    return c


def _step(name, **kw):
    # the 8B-shaped layer: d = 4096, 32 heads x 128, SwiGLU 12288, vocabulary
    # 126464; n_view is the view's token count, `level` how coarse it is (it
    # sets the spread of its values), masked the response positions still open
    c = dict(kind="step", dtype="f16", layers=1, d=4096, ffn=12288,
             vocab=126464, tiled=True, seqs=1, mix=0, level=2, n_view=729,
             prompt=32, resp=128, masked=32)
    c.update(kw, name=name)
    return c


def listed():
    return [
        # one 27 x 27 crop into its pooled levels: the start of every request,
        # and the smallest call
        _views("views-pool-1crop"),
        # five crops, the prune realizer: keys, decisions, kept rows
        _views("views-prune-5crops", realizer="prune", crops=5),
        # four crops, the merge realizer: edge similarities, single linkage,
        # group means
        _views("views-merge-4crops", realizer="merge", crops=4),
        # the end of a step of a batch of 16: commit two positions of each
        # response and allocate the next step's evidence
        dict(name="commit-16", kind="commit", seqs=16, resp=128, k=2, K=3,
             masked=90),
        # the tiny fp32 model's whole loop under the policy: 8 steps, latency
        # and launches
        dict(name="loop-tiny-f32", kind="loop", d=256, heads=4, ffn=1024,
             vocab=1024, layers=2, grid=12, crops=1, prompt=16, resp=32, T=8,
             k=4),
        # one layer at the coarsest view of one crop (49 tokens), most of the
        # response committed: the most frequent step of a loop
        _step("step-209", n_view=49, level=0),
        # one crop in full, early in a loop
        _step("step-889", masked=112),
        # a bf16 model of half the width with two layers and a row-major head:
        # other sizes than the 8B ones, the other operand format
        _step("step-bf16-half", dtype="bf16", layers=2, d=2048, ffn=5632,
              vocab=32003, tiled=False, masked=64),
        # five crops in full and a 256-token response, one layer
        _step("step-3965", n_view=3645, prompt=64, resp=256, masked=64),
        # the 8B-shaped stack at two of its three views of four crops (eight
        # of its 32 equal layers, so that weights can be made many times)
        _step("stack-372", layers=8, n_view=196, level=0, prompt=48),
        _step("stack-3092", layers=8, n_view=2916, prompt=48),
        # sixteen requests in one step, each with its own crops, level and
        # prompt
        _step("batch-16", seqs=16, mix=5, n_view=3645, prompt=96),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["views", "views", "commit", "loop", "step", "step",
                       "step", "stack", "batch", "other"])
    if kind == "views":
        r = rng.choice(["pool", "mixed", "prune", "merge"])
        return dict(kind="views", realizer=r, crops=rng.randint(1, 5),
                    dtype=rng.choice(["f16", "f16", "bf16", "f32"]),
                    grid=rng.randint(9, 32), d=8 * log_int(32, 512),
                    K=3 if r == "mixed" else rng.choice([2, 3, 3, 4]),
                    stride=rng.randint(2, 4) if r == "mixed" else 0)
    if kind == "commit":
        resp = log_int(24, 1024)
        return dict(kind="commit", seqs=log_int(1, 64), resp=resp,
                    k=rng.randint(1, 8), K=rng.randint(2, 4),
                    masked=rng.randint(9, resp))
    if kind == "loop":
        k = rng.randint(2, 5)
        T = rng.randint(4, 8)
        heads = rng.randint(2, 6)
        return dict(kind="loop", d=64 * heads, heads=heads,
                    ffn=rng.randint(200, 1200), vocab=rng.randint(300, 2100),
                    layers=rng.randint(1, 3), grid=rng.randint(6, 14),
                    crops=rng.randint(1, 2), prompt=rng.randint(2, 24),
                    resp=k * T + rng.randint(0, 16), T=T, k=k)
    resp = rng.choice([64, 96, 128, 128, 200, 256])
    c = dict(kind="step", dtype=rng.choice(["f16", "f16", "bf16"]), layers=1,
             d=4096, ffn=12288, vocab=126464, tiled=rng.random() < 0.75,
             seqs=1, mix=0, prompt=rng.randint(32, 96), resp=resp,
             masked=log_int(2, resp), level=rng.randint(0, 2))
    side = (27 + (1 << (2 - c["level"])) - 1) >> (2 - c["level"])
    c["n_view"] = rng.randint(1, 5) * side * side
    if kind == "stack":
        c.update(dtype="f16", layers=rng.randint(2, 8))
    elif kind == "batch":
        c.update(seqs=rng.randint(2, 16), mix=rng.randint(1, 999), resp=128,
                 masked=log_int(2, 64), level=2,
                 n_view=729 * rng.randint(1, 5))
    elif kind == "other":
        c.update(layers=2, d=128 * rng.randint(4, 24),
                 ffn=64 * rng.randint(16, 150), vocab=rng.randint(4000, 60000))
    # no dearer than the largest listed case
    for key in ("seqs", "layers"):
        while c[key] > 1 and work(c)["flops"] > 1e13:
            c[key] -= 1
    return c


# ------------------------------------------------------------------ shapes --

def _sides(c):
    """Window counts per side of each level of a crop."""
    return [-(-c["grid"] // (1 << (c["K"] - 1 - lv))) for lv in range(c["K"])]


def _lattice(c):
    return range(c["stride"] // 2, c["grid"], c["stride"])


def _level_sizes(c):
    n = [c["crops"] * w * w for w in _sides(c)]
    if c["realizer"] == "mixed":
        n[1] = n[0] + c["crops"] * len(_lattice(c)) ** 2
    return n


def _seq_shapes(c):
    """(view tokens, level, prompt length) of each sequence of a step."""
    if c["seqs"] == 1:
        return [(c["n_view"], c["level"], c["prompt"])]
    rng, out = random.Random(c["mix"]), []
    for _ in range(c["seqs"]):
        lv = rng.choice([0, 1, 2, 2])
        side = (7, 14, 27)[lv]
        out.append((rng.randint(1, c["n_view"] // 729) * side * side, lv,
                    rng.randint(min(32, c["prompt"]), c["prompt"])))
    return out


def work(c):
    if c["kind"] == "views":
        es = 4 if c["dtype"] == "f32" else 2
        n = c["crops"] * c["grid"] ** 2 + sum(_level_sizes(c)[:-1])
        return {"bytes": n * c["d"] * es, "flops": c["crops"] * c["grid"] ** 2 * c["d"]}
    if c["kind"] == "commit":
        return {"bytes": c["seqs"] * c["resp"] * 18, "flops": 0}
    if c["kind"] == "loop":
        d, F = c["d"], c["ffn"]
        flops = bytes_ = 0
        sides = [-(-c["grid"] // 4), -(-c["grid"] // 2), c["grid"]]
        n = c["crops"] * sides[1] ** 2 + c["prompt"] + c["resp"]
        for t in range(c["T"]):
            rows = c["resp"] - c["k"] * t
            flops += c["layers"] * (2 * n * (4 * d * d + 3 * d * F) + 4 * n * n * d)
            flops += 2 * rows * d * c["vocab"]
            bytes_ += 4 * (c["layers"] * (4 * d * d + 3 * d * F) + d * c["vocab"] + n * d)
        return {"bytes": bytes_, "flops": flops}
    d, F, V = c["d"], c["ffn"], c["vocab"]
    rows = c["seqs"] * c["masked"]
    flops = 2.0 * rows * d * V
    tokens = 0
    for nv, _, p in _seq_shapes(c):
        n = nv + p + c["resp"]
        tokens += n
        flops += c["layers"] * 4.0 * n * n * d
    flops += c["layers"] * 2.0 * tokens * (4 * d * d + 3 * d * F)
    weights = 2.0 * (c["layers"] * (4 * d * d + 3 * d * F) + d * V)
    return {"bytes": weights + 2.0 * tokens * d + 4.0 * rows * V, "flops": flops}


def tolerance(c):
    if c["kind"] in ("views", "commit"):
        # decisions and copies; means summed in 64 bits and rounded once
        return "exact"
    if c["kind"] == "loop":
        # 32-bit sums in another order, a few layers deep
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    # 16-bit operands: one rounding of every activation tensor of every layer
    rel = (3e-3 if c["dtype"] == "f16" else 2e-2) * math.sqrt(c["layers"])
    return {"rel": min(rel, 3e-2), "max": min(12 * rel, 0.9)}


# ------------------------------------------------------------------ inputs --

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + stream)
    return g


def _normal(g, shape, std, dtype, model=torch.bfloat16):
    """Values of a bf16 model (its weights and encodings), in `dtype`."""
    t = torch.randn(shape, generator=g, device="cuda",
                    dtype=torch.float32 if dtype == torch.float32 else model)
    return t.mul_(std).to(dtype)


def _layer(c, seed, i, dtype):
    d, F = c["d"], c["ffn"]
    g = _gen(seed, 100 + i)
    shapes = dict(wqkv=(3 * d, d), wo=(d, d), wg=(F, d), wu=(F, d), wd=(d, F))
    return {k: _normal(g, s, 0.02, dtype) for k, s in shapes.items()}


def _tables(c, seed, dtype):
    g = _gen(seed, 50)
    return (_normal(g, (c["vocab"], c["d"]), 0.02, dtype),
            _normal(g, (c["vocab"], c["d"]), 0.02, dtype))


def _visual(c, seed):
    """Encodings of image crops: neighbouring tokens are alike (a coarse
    field), each with detail of its own."""
    g, G = _gen(seed, 1), c["grid"]
    lo = torch.randn((c["crops"], c["d"], -(-G // 3), -(-G // 3)), generator=g,
                     device="cuda")
    v = torch.nn.functional.interpolate(lo, size=(G, G), mode="bilinear",
                                        align_corners=False)
    v = v + 0.6 * torch.randn(v.shape, generator=g, device="cuda")
    v = v.permute(0, 2, 3, 1).reshape(c["crops"] * G * G, c["d"])
    return v.to(torch.bfloat16).to(DTYPES[c["dtype"]][0]).contiguous()


def _open_rows(c, g):
    """[seqs, resp] flags with `masked` open positions each, at random."""
    order = torch.rand((c["seqs"], c["resp"]), generator=g, device="cuda").argsort(1)
    return (order < c["masked"]).to(torch.uint8)


def _step_inputs(c, seed):
    dtype = DTYPES[c["dtype"]][0]
    shapes = _seq_shapes(c)
    g = _gen(seed, 2)
    views = [_normal(g, (nv, c["d"]), 0.25 * (1 << lv), dtype)
             for nv, lv, _ in shapes]
    cu = [0]
    for _, _, p in shapes:
        cu.append(cu[-1] + p)
    prompt = torch.randint(0, c["vocab"] - 1, (cu[-1],), generator=g,
                           device="cuda", dtype=torch.int32)
    masked = _open_rows(c, g)
    ids = torch.randint(0, c["vocab"] - 1, (c["seqs"], c["resp"]), generator=g,
                        device="cuda", dtype=torch.int32)
    ids = torch.where(masked.bool(), c["vocab"] - 1, ids).to(torch.int32)
    return dict(views=views, n_view=[s[0] for s in shapes], cu=cu,
                prompt=prompt, masked=masked.reshape(-1), ids=ids.reshape(-1))


def _loop_weights(c, seed):
    embed, head = _tables(c, seed, torch.float32)
    return embed, head, [_layer(c, seed, i, torch.float32)
                         for i in range(c["layers"])]


# the policy's settings (the LLaDA-V defaults with a grounding demand)
POLICY = dict(B=0.75, rho=0.20, alpha=1.0, demand=0.824, early=1)


def _policy(K):
    p = POLICY
    return dv.Policy(p["B"], p["rho"], p["alpha"], p["demand"], p["early"], K)


def prepare(c, seed):
    with torch.no_grad():
        return globals()["_prepare_" + c["kind"]](c, seed)


def _prepare_views(c, seed):
    geom = dv.ViewGeom(c["crops"], c["grid"], c["d"], c["K"],
                       DTYPES[c["dtype"]][1], c["stride"],
                       REALIZERS[c["realizer"]])
    v = _visual(c, seed)
    levels = [torch.empty((n, c["d"]), dtype=v.dtype, device="cuda")
              for n in dv.davet_view_sizes(geom)[:-1]]
    nb = dv.davet_views_scratch_bytes(geom)
    scratch = torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None
    return dict(c=c, geom=geom, v=v, levels=levels, scratch=scratch)


def _prepare_commit(c, seed):
    g = _gen(seed, 3)
    n, L = c["seqs"], c["resp"]
    masked = _open_rows(c, g)
    conf = torch.rand((n, L), generator=g, device="cuda")
    conf = torch.where(masked.bool(), conf, -math.inf).reshape(-1)
    am, prev, ids = (torch.randint(0, 126463, (n * L,), generator=g,
                                   device="cuda", dtype=torch.int32)
                     for _ in range(3))
    same = torch.rand(n * L, generator=g, device="cuda") < 0.8
    prev = torch.where(same, am, prev)
    pols = [_policy(c["K"]) for _ in range(n)]
    lo, up = dv.davet_policy_envelope(pols[0], 64)
    i32 = dict(dtype=torch.int32, device="cuda")
    f64 = dict(dtype=torch.float64, device="cuda")
    return dict(c=c, conf=conf, am=am, prev=prev, pols=pols,
                lower=np.asarray(lo * n), upper=np.asarray(up * n),
                masked0=masked.reshape(-1), ids0=ids,
                masked=masked.reshape(-1).clone(), ids=ids.clone(),
                selected=torch.empty((n, c["k"]), **i32),
                level=torch.empty(n, **i32), budget=torch.empty(n, **f64),
                risk=torch.empty(n, **f64))


def _prepare_loop(c, seed):
    embed, head, layers = _loop_weights(c, seed)
    vc = dict(c, dtype="f32", K=3, stride=0)
    geom = dv.ViewGeom(c["crops"], c["grid"], c["d"], 3, dv.DAVET_F32)
    cfg = dv.ModelCfg(c["layers"], c["d"], c["heads"], c["d"] // c["heads"],
                      c["ffn"], c["vocab"], c["vocab"] - 1, EPS, THETA,
                      dv.DAVET_F32)
    sizes = dv.davet_view_sizes(geom)
    tokens = sizes[2] + c["prompt"] + c["resp"]
    f32, i32 = dict(device="cuda"), dict(dtype=torch.int32, device="cuda")
    prompt = torch.randint(0, c["vocab"] - 1, (c["prompt"],),
                           generator=_gen(seed, 2), **i32)
    return dict(
        c=c, cfg=cfg, geom=geom, W=dv.Weights(embed, head, layers),
        v=_visual(vc, seed), prompt=prompt, pols=[_policy(3)],
        levels=[torch.empty((n, c["d"]), **f32) for n in sizes[:2]],
        ids=torch.empty(c["resp"], **i32),
        masked=torch.empty(c["resp"], dtype=torch.uint8, device="cuda"),
        conf=torch.empty((c["T"], c["resp"]), **f32),
        argmax=torch.empty((c["T"], c["resp"]), **i32),
        mailbox=dv.default_mailbox(),
        ws=torch.empty(dv.davet_workspace_bytes(cfg, tokens, 1, c["resp"]),
                       dtype=torch.uint8, device="cuda"))


def _prepare_step(c, seed):
    dtype, code = DTYPES[c["dtype"]]
    embed, head = _tables(c, seed, dtype)
    if c["tiled"]:
        packed = torch.empty(dv.davet_head_tiled_elems(c["vocab"], c["d"]),
                             dtype=dtype, device="cuda")
        dv.davet_pack_head(head, packed, c["vocab"], c["d"], code)
        head = packed
    layers = [_layer(c, seed, i, dtype) for i in range(c["layers"])]
    cfg = dv.ModelCfg(c["layers"], c["d"], c["d"] // 128, 128, c["ffn"],
                      c["vocab"], c["vocab"] - 1, EPS, THETA, code)
    s = _step_inputs(c, seed)
    rows = c["seqs"] * c["resp"]
    tokens = sum(s["n_view"]) + s["cu"][-1] + rows
    s.update(
        c=c, cfg=cfg,
        W=dv.Weights(embed, head, layers, None,
                     dv.DAVET_HEAD_TILED if c["tiled"] else dv.DAVET_HEAD_ROWS),
        conf=torch.empty(rows, device="cuda"),
        argmax=torch.empty(rows, dtype=torch.int32, device="cuda"),
        # rows of committed positions are not written
        logits=torch.zeros((rows, c["vocab"]), device="cuda"),
        ws=torch.empty(dv.davet_workspace_bytes(cfg, tokens, c["seqs"], c["resp"]),
                       dtype=torch.uint8, device="cuda"))
    return s


# --------------------------------------------------------------------- run --

def run(s):
    return globals()["_run_" + s["c"]["kind"]](s)


def _run_views(s):
    dv.davet_build_views(s["geom"], s["v"], s["levels"], scratch=s["scratch"])
    return s["levels"]


def _run_commit(s):
    c = s["c"]
    s["masked"].copy_(s["masked0"])
    s["ids"].copy_(s["ids0"])
    dv.davet_unmask(c["seqs"], c["resp"], c["k"], s["conf"], s["am"], s["ids"],
                    s["masked"], s["selected"])
    dv.davet_policy_step_device(s["pols"], 20, 64, s["lower"], s["upper"],
                                s["conf"], s["am"], s["prev"], s["masked"],
                                s["level"], s["budget"], s["risk"])
    return {k: s[k] for k in ("ids", "masked", "selected", "level", "budget",
                              "risk")}


def _run_loop(s):
    c = s["c"]
    s["ids"].fill_(c["vocab"] - 1)
    s["masked"].fill_(1)
    levels, budgets = dv.davet_run_schedule(
        s["cfg"], s["W"], [s["geom"]], [s["v"]], s["levels"], s["prompt"],
        [0, c["prompt"]], c["resp"], c["T"], c["k"], s["pols"], None, s["ids"],
        s["masked"], s["ws"], s["conf"], s["argmax"], mailbox=s["mailbox"])
    return {"conf": s["conf"], "argmax": s["argmax"], "ids": s["ids"],
            "masked": s["masked"], "levels": torch.tensor(levels),
            "budgets": torch.tensor(budgets, dtype=torch.float64),
            "views": s["levels"]}


def _run_step(s):
    dv.davet_denoise_step(s["cfg"], s["W"], s["views"], s["n_view"],
                          s["prompt"], s["cu"], s["ids"], s["masked"],
                          s["c"]["resp"], s["conf"], s["argmax"], s["logits"],
                          s["ws"])
    return {"logits": s["logits"], "conf": s["conf"]}


# ------------------------------------------------- the same in 64 bits -----

def exact(c, seed):
    with torch.no_grad():
        return globals()["_exact_" + c["kind"]](c, seed)


def _norm(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)


def _rope(x, n, heads, hd):
    half = hd // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / hd)
    a = torch.arange(n, dtype=torch.float64, device="cuda")[:, None] * inv
    cos, sin = a.cos()[:, None], a.sin()[:, None]
    x = x.reshape(n, heads, hd)
    p, q = x[..., :half], x[..., half:]
    return torch.cat([p * cos - q * sin, q * cos + p * sin], -1)


def _layer64(x, w, spans, heads):
    d = x.shape[1]
    hd = d // heads
    qkv = _norm(x) @ w["wqkv"].double().T
    o = torch.empty_like(x)
    for a, b in spans:
        n = b - a
        q = _rope(qkv[a:b, :d], n, heads, hd)
        k = _rope(qkv[a:b, d:2 * d], n, heads, hd)
        v = qkv[a:b, 2 * d:].reshape(n, heads, hd)
        for h in range(heads):
            p = torch.softmax(q[:, h] @ k[:, h].T / math.sqrt(hd), -1)
            o[a:b, h * hd:(h + 1) * hd] = p @ v[:, h]
    x = x + o @ w["wo"].double().T
    y = _norm(x)
    for i in range(0, x.shape[0], 4096):          # bounds the memory
        h = torch.nn.functional.silu(y[i:i + 4096] @ w["wg"].double().T)
        h *= y[i:i + 4096] @ w["wu"].double().T
        x[i:i + 4096] += h @ w["wd"].double().T
    return x


def _decode64(hidden, head, mask_id):
    logits = _norm(hidden) @ head.double().T
    l = logits.clone()
    l[:, mask_id] = -math.inf
    conf, am = torch.softmax(l, -1).max(-1)
    return logits, conf, am


def _exact_step(c, seed):
    embed, head = _tables(c, seed, DTYPES[c["dtype"]][0])
    s = _step_inputs(c, seed)
    L, parts, spans, at = c["resp"], [], [], 0
    for i, v in enumerate(s["views"]):
        ids = torch.cat([s["prompt"][s["cu"][i]:s["cu"][i + 1]],
                         s["ids"][i * L:(i + 1) * L]]).long()
        parts += [v.double(), embed[ids].double()]
        spans.append((at, at + v.shape[0] + len(ids)))
        at = spans[-1][1]
    x = torch.cat(parts)
    for i in range(c["layers"]):
        x = _layer64(x, _layer(c, seed, i, DTYPES[c["dtype"]][0]), spans,
                     c["d"] // 128)
    rows = torch.cat([x[b - L:b] for _, b in spans])
    open_ = s["masked"].bool()
    at = open_.nonzero()[:, 0]
    logits = torch.zeros((len(rows), c["vocab"]), device="cuda")
    conf = torch.full((len(rows),), -math.inf, dtype=torch.float64, device="cuda")
    for i in range(0, len(at), 128):
        j = at[i:i + 128]
        lg, cf, _ = _decode64(rows[j], head, c["vocab"] - 1)
        # kept in 32 bits: two gigabytes less, far below 16-bit errors
        logits[j], conf[j] = lg.float(), cf
    return {"logits": logits, "conf": conf}


def _windows(c):
    """Window side of each level below the finest."""
    return [1 << (c["K"] - 1 - lv) for lv in range(c["K"] - 1)]


def _pool_level64(v, c, f):
    G = c["grid"]
    x = v.double().reshape(c["crops"], G, G, -1)
    W = -(-G // f)
    rows = []
    for i in range(W):
        for j in range(W):
            w = x[:, i * f:(i + 1) * f, j * f:(j + 1) * f]
            rows.append(w.reshape(c["crops"], -1, w.shape[-1]).mean(1))
    return torch.stack(rows, 1)                       # [crops, W * W, d]


def _exact_views(c, seed):
    v = _visual(c, seed)
    G, d = c["grid"], c["d"]
    counts = [(-(-G // f)) ** 2 for f in _windows(c)]
    if c["realizer"] in ("pool", "mixed"):
        lv = [_pool_level64(v, c, f) for f in _windows(c)]
        if c["realizer"] == "mixed":
            x = v.double().reshape(c["crops"], G, G, d)
            at = list(_lattice(c))
            lv[1] = torch.cat([lv[0], x[:, at][:, :, at].reshape(c["crops"], -1, d)], 1)
        return [x.reshape(-1, d) for x in lv]
    out = [[] for _ in counts]
    for crop in v.double().reshape(c["crops"], G * G, d):
        if c["realizer"] == "prune":
            order = crop.abs().sum(1).sort(descending=True, stable=True)[1]
            for n, o in zip(counts, out):
                o.append(crop[order[:n].sort()[0]])
            continue
        g = crop.reshape(G, G, d)
        nn = (crop * crop).sum(1).reshape(G, G)
        right = (g[:, 1:] * g[:, :-1]).sum(-1) / torch.sqrt(nn[:, 1:] * nn[:, :-1])
        down = (g[1:] * g[:-1]).sum(-1) / torch.sqrt(nn[1:] * nn[:-1])
        ends = [(r * G + s, r * G + s + 1) for r in range(G) for s in range(G - 1)]
        ends += [(r * G + s, (r + 1) * G + s) for r in range(G - 1) for s in range(G)]
        keys = torch.cat([right.reshape(-1), down.reshape(-1)]).cpu()
        root = list(range(G * G))

        def find(a):
            while root[a] != a:
                a = root[a]
            return a

        groups, level = G * G, len(counts) - 1
        for e in [-1] + keys.sort(descending=True, stable=True)[1].tolist():
            if e >= 0:
                a, b = (find(x) for x in ends[e])
                if a == b:
                    continue
                root[max(a, b)] = min(a, b)
                groups -= 1
            while level >= 0 and groups == counts[level]:
                own = torch.tensor([find(i) for i in range(G * G)], device="cuda")
                ids, at = own.unique(return_inverse=True)
                sums = torch.zeros((len(ids), d), dtype=torch.float64, device="cuda")
                sums.index_add_(0, at, crop)
                out[level].append(sums / at.bincount()[:, None])
                level -= 1
    return [torch.cat(o) for o in out]


def _scaled(p, beta):
    """min(1, s p) with mean beta."""
    if beta >= 1 or beta <= 0:
        return [float(beta >= 1)] * len(p)
    for j, big in enumerate(sorted(p, reverse=True)):
        s = (len(p) * beta - j) / sum(sorted(p, reverse=True)[j:])
        if s * big <= 1:
            return [min(1.0, s * x) for x in p]
    return [1.0] * len(p)


def _allocate(t, T, cbar, churn, K):
    """(budget, level, risk) of step t from the signals of step t - 1."""
    P = POLICY
    p = [1 - (i + 0.5) / T for i in range(T)]
    lo = _scaled(p, (1 - P["rho"]) * P["B"])[t - 1]
    up = _scaled(p, (1 - P["rho"] + P["rho"] * P["demand"]) * P["B"])[t - 1]
    r = 1.0 if t == 1 else 1 - P["alpha"] * cbar * (1 - churn)
    b = lo + r * (up - lo)
    return b, sum(j / K <= b for j in range(1, K)), r


def _signals(conf, am, prev, masked):
    m = masked.bool()
    n = int(m.sum())
    cbar = float(conf[m].double().sum()) / n if n else 0.0
    churn = float((am[m] != prev[m]).sum()) / n if n and prev is not None else 0.0
    return cbar, churn


def _exact_commit(c, seed):
    s = _prepare_commit(c, seed)
    L, out = c["resp"], dict(ids=[], masked=[], selected=[], level=[], budget=[], risk=[])
    for i in range(c["seqs"]):
        sl = slice(i * L, (i + 1) * L)
        conf, am, m, ids = (s[k][sl].clone() for k in ("conf", "am", "masked0", "ids0"))
        sel = conf.sort(descending=True, stable=True)[1][:min(c["k"], c["masked"])]
        ids[sel], m[sel] = am[sel], 0
        b, lv, r = _allocate(21, 64, *_signals(conf, am, s["prev"][sl], m), c["K"])
        pad = torch.full((c["k"] - len(sel),), -1, device="cuda")
        for k, x in zip(out, (ids, m, torch.cat([sel, pad]), lv, b, r)):
            out[k].append(x)
    f64 = dict(dtype=torch.float64)
    return dict(ids=torch.cat(out["ids"]), masked=torch.cat(out["masked"]),
                selected=torch.stack(out["selected"]),
                level=torch.tensor(out["level"]),
                budget=torch.tensor(out["budget"], **f64),
                risk=torch.tensor(out["risk"], **f64))


def _exact_loop(c, seed):
    embed, head, layers = _loop_weights(c, seed)
    vc = dict(c, dtype="f32", K=3, stride=0)
    v = _visual(vc, seed)
    prompt = _prepare_loop(c, seed)["prompt"].long()
    views = [_pool_level64(v, vc, f).reshape(-1, c["d"]) for f in (4, 2)]
    views.append(v.double())
    L, T, mask_id = c["resp"], c["T"], c["vocab"] - 1
    ids = torch.full((L,), mask_id, device="cuda")
    masked = torch.ones(L, dtype=torch.uint8, device="cuda")
    cbar = churn = 0.0
    prev, trace = None, dict(conf=[], argmax=[], levels=[], budgets=[])
    for t in range(1, T + 1):
        b, lv, _ = _allocate(t, T, cbar, churn, 3)
        x = torch.cat([views[lv], embed[prompt].double(), embed[ids].double()])
        for w in layers:
            x = _layer64(x, w, [(0, len(x))], c["heads"])
        _, cf, a = _decode64(x[len(x) - L:], head, mask_id)
        conf = torch.where(masked.bool(), cf, -math.inf)
        am = torch.where(masked.bool(), a, -1)
        sel = conf.sort(descending=True, stable=True)[1][:min(c["k"], int(masked.sum()))]
        ids[sel], masked[sel] = am[sel], 0
        cbar, churn = _signals(conf, am, prev, masked)
        prev = am
        for k, x in zip(trace, (conf, am, lv, b)):
            trace[k].append(x)
    return {"conf": torch.stack(trace["conf"]),
            "argmax": torch.stack(trace["argmax"]), "ids": ids,
            "masked": masked, "levels": torch.tensor(trace["levels"]),
            "budgets": torch.tensor(trace["budgets"], dtype=torch.float64),
            "views": views[:2]}
