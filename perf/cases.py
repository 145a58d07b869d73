"""The work a rollout program has this library do, as cases that can be timed.

Kinds of case:

* ``decode``: one ``Context.tree_decode`` over a finished forest -- every
  leaf's new query against its whole chain.
* ``step``: one step of segment-level decoding with device-resident lengths:
  ``Context.kv_append`` of one token per leaf, then ``Context.tree_decode``.
  When the segments are full the program opens its cache anew at the point of
  the last fork, so passes stay alike.
* ``prefill``: ``Context.prefill`` of new prompts, or of segments that
  continue a prompt already in the cache, into fresh nodes.  The pools have
  room for some batches; when they are full the program opens a new context
  over them.
* ``advantage``: ``Context.tree_advantage`` of every decoded trajectory.
* ``rollout``: a whole small rollout: prompts prefilled, paths forked before
  every segment, each segment decoded token by token.

Trees have the shapes of TreePO rollouts: prompts as roots, segments of at
most ``seg`` tokens, binary forks at the first boundaries and unbranched
growth after them ("binary"), or random forks and early stops ("irregular").
Keys, values and queries are N(0, 1) in bf16, rewards 0 or 1.
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2508_17445_amd import Context

DEVICE = "cuda"
BATCHES = 32        # prefill batches (and rollouts) the pools of a state hold
STEP_SETS = 16      # different token / query sets a decode loop cycles through

# (query heads, KV heads, head dim): the 7B-style GQA shape, a wider one, the
# small test shape and the head-dim-64 and one-query-per-KV-head variants.
SHAPES = ((28, 4, 128), (40, 8, 128), (4, 1, 64), (16, 2, 64), (32, 4, 64), (8, 8, 128), (12, 2, 64))


def _heads(i):
    hq, hkv, d = SHAPES[i]
    return {"hq": hq, "hkv": hkv, "d": d}


def listed():
    return [
        # One 64-token prompt, 16-token segments, three binary forks: the
        # smallest tree, where launches and latency are all there is.
        {"name": "decode_tiny", "kind": "decode", "shape": "binary", "prompts": 1, "prompt_lo": 64, "prompt_hi": 64,
         "seg": 16, "levels": 3, "total_lo": 112, "total_hi": 112, "block": 16, "shape_seed": 1, **_heads(2)},
        # One prompt, 16 leaves of 7,680 tokens: an ordinary tree of a long
        # reasoning rollout.
        {"name": "decode_tree16", "kind": "decode", "shape": "binary", "prompts": 1, "prompt_lo": 512,
         "prompt_hi": 512, "seg": 512, "levels": 4, "total_lo": 7680, "total_hi": 7680, "block": 64, "shape_seed": 2,
         **_heads(0)},
        # The same tree at head dim 64.
        {"name": "decode_tree16_d64", "kind": "decode", "shape": "binary", "prompts": 1, "prompt_lo": 512,
         "prompt_hi": 512, "seg": 512, "levels": 4, "total_lo": 7680, "total_hi": 7680, "block": 64, "shape_seed": 2,
         **_heads(3)},
        # 32 prompts whose paths fork 1 to 4 ways and stop early: ragged
        # lengths everywhere, many small nodes.
        {"name": "decode_irregular", "kind": "decode", "shape": "irregular", "prompts": 32, "prompt_lo": 512,
         "prompt_hi": 512, "seg": 256, "levels": 0, "total_lo": 8192, "total_hi": 8192, "block": 64, "shape_seed": 4,
         **_heads(0)},
        # A training batch: 64 prompts of 256 to 1,024 tokens, 16 ragged
        # leaves each.
        {"name": "decode_batch", "kind": "decode", "shape": "binary", "prompts": 64, "prompt_lo": 256,
         "prompt_hi": 1024, "seg": 512, "levels": 4, "total_lo": 2561, "total_hi": 8192, "block": 64, "shape_seed": 3,
         **_heads(0)},
        # Segment-level decoding of the 16-leaf tree, one token per pass.
        {"name": "step_tree16", "kind": "step", "shape": "binary", "prompts": 1, "prompt_lo": 512, "prompt_hi": 512,
         "seg": 512, "levels": 4, "total_lo": 7168, "total_hi": 7168, "block": 64, "shape_seed": 2, **_heads(0)},
        # Long contexts: 8 prompts, 32 leaves each of about 16,000 tokens; the
        # largest decode, one token per pass.
        {"name": "step_long", "kind": "step", "shape": "binary", "prompts": 8, "prompt_lo": 2048, "prompt_hi": 2048,
         "seg": 1024, "levels": 5, "total_lo": 15360, "total_hi": 15360, "block": 64, "shape_seed": 5, **_heads(1)},
        # One prompt of 513 tokens (a ragged last tile): a request that
        # arrives alone.
        {"name": "prefill_one", "kind": "prefill", "rows": 1, "new_lo": 513, "new_hi": 513, "prefix": 0, "block": 64,
         "shape_seed": 6, **_heads(0)},
        # The training batch's prompts in one call.
        {"name": "prefill_batch", "kind": "prefill", "rows": 64, "new_lo": 256, "new_hi": 1024, "prefix": 0,
         "block": 64, "shape_seed": 3, **_heads(0)},
        # Long prompts of the wide model.
        {"name": "prefill_long", "kind": "prefill", "rows": 8, "new_lo": 2048, "new_hi": 2048, "prefix": 0,
         "block": 64, "shape_seed": 5, **_heads(1)},
        # The advantages of the training batch's 1,024 trajectories.
        {"name": "advantage_batch", "kind": "advantage", "shape": "binary", "prompts": 64, "prompt_lo": 256,
         "prompt_hi": 1024, "seg": 512, "levels": 4, "total_lo": 2561, "total_hi": 8192, "block": 64, "shape_seed": 3,
         "weighting": 0, **_heads(0)},
        # A whole small rollout: 4 prompts, three binary forks, 16-token
        # segments: prefill, forks, plans and 48 decode steps.
        {"name": "rollout_small", "kind": "rollout", "prompts": 4, "new_lo": 200, "new_hi": 500, "levels": 3,
         "seg": 16, "block": 16, "shape_seed": 7, **_heads(0)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "step", "step", "prefill", "prefill", "prefill", "advantage",
                       "rollout"])
    heads = _heads(rng.choice([0, 0, 0, 1, 2, 3, 4, 5, 6]))
    seed = rng.randrange(1 << 20)
    block = rng.choice([16, 32, 64, 64])
    if kind == "prefill":
        rows = _log_int(rng, 1, 64)
        hi = _log_int(rng, 17, 2048)
        # at most the query rows and half the key-value products of the largest listed one
        while rows * hi > 40000 or rows * hi * hi * heads["hq"] > 8 * 2048 * 2048 * 40:
            hi = max(1, hi // 2)
        lo = max(1, int(hi * rng.uniform(0.25, 1.0)))
        prefix = rng.choice([0, 0, _log_int(rng, 33, 1500)])
        if rows * hi * (hi + 2 * prefix) * heads["hq"] > 8 * 2048 * 2048 * 40:
            prefix = 0
        return {"kind": kind, "rows": rows, "new_lo": lo, "new_hi": hi, "prefix": prefix, "block": block,
                "shape_seed": seed, **heads}
    if kind == "rollout":
        return {"kind": kind, "prompts": rng.randint(1, 4), "new_lo": 40, "new_hi": _log_int(rng, 64, 500),
                "levels": rng.randint(1, 3), "seg": rng.randint(5, 16), "block": block, "shape_seed": seed, **heads}
    while True:
        seg = _log_int(rng, 16, 1024)
        prompts = _log_int(rng, 1, 64)
        plo = _log_int(rng, 32, 1024)
        phi = plo + rng.randrange(plo)
        c = {"kind": kind, "prompts": prompts, "prompt_lo": plo, "prompt_hi": phi, "seg": seg, "block": block,
             "shape_seed": seed, **heads}
        if kind == "advantage":
            c["weighting"] = rng.randint(0, 1)
        if rng.random() < 0.3 and kind != "step":
            total = phi + seg * rng.randint(2, 24)
            c.update(shape="irregular", levels=0, total_lo=total, total_hi=total)
        else:
            levels = rng.randint(0, 5)
            lo = phi + levels * seg + 1
            hi = lo + _log_int(rng, 1, 12000)
            c.update(shape="binary", levels=levels, total_lo=lo, total_hi=hi)
        if c["total_hi"] > 16384 or prompts << c["levels"] > 1024:
            continue
        f = _forest(c)
        kv_bytes = sum(f["len"]) * c["hkv"] * c["d"] * 4
        if kv_bytes <= 7 << 30 and len(f["len"]) <= 12000 and len(f["leaves"]) <= 1024:
            return c


# ---- trees --------------------------------------------------------------------


def _forest(c):
    """Nodes in creation order (parents first): parent, tokens, capacity, and
    the leaves to decode (a step's leaves are fresh, empty segments)."""
    r = random.Random(c["shape_seed"])
    seg = c["seg"]
    parent, length, cap, start, depth = [], [], [], [], []

    def node(p, n, cp):
        parent.append(p)
        length.append(n)
        cap.append(cp)
        start.append(0 if p < 0 else start[p] + length[p])
        depth.append(0 if p < 0 else depth[p] + 1)
        return len(parent) - 1

    def end(i):
        return start[i] + length[i]

    roots = []
    for _ in range(c["prompts"]):
        n = r.randint(c["prompt_lo"], c["prompt_hi"])
        roots.append(node(-1, n, n))
    if c["shape"] == "binary":
        front = [(x, None) for x in roots]
        for lv in range(c["levels"]):
            last = lv == c["levels"] - 1
            nxt = []
            for x, _ in front:
                for _ in range(2):
                    total = r.randint(c["total_lo"], c["total_hi"]) if last else None
                    nxt.append((node(x, seg if total is None else max(1, min(seg, total - end(x))), seg), total))
            front = nxt
        front = [(x, r.randint(c["total_lo"], c["total_hi"]) if t is None else t) for x, t in front]
        leaves = [x for x, _ in front]
        grow = [(k, t) for k, (_, t) in enumerate(front)]
        while grow:
            nxt = []
            for k, t in grow:
                x = leaves[k]
                if end(x) < t:
                    leaves[k] = node(x, min(seg, t - end(x)), seg)
                    nxt.append((k, t))
            grow = nxt
    else:
        count = {x: 1 for x in roots}
        front = [(x, x) for x in roots]
        kids = set()
        while front:
            nxt = []
            for x, root in front:
                br = min(r.randint(1, 4), 32 - count[root] + 1)
                count[root] += br - 1
                for _ in range(br):
                    avail = min(seg, c["total_hi"] - end(x))
                    stop = r.random() < 0.2
                    n = r.randint(1, avail) if stop else avail
                    y = node(x, n, seg)
                    kids.add(x)
                    if not stop and end(y) < c["total_hi"]:
                        nxt.append((y, root))
            front = nxt
        leaves = [i for i in range(len(parent)) if i not in kids]
    if c["kind"] == "step":
        leaves = [node(x, 0, seg) for x in leaves]
    return {"parent": parent, "len": length, "cap": cap, "leaves": leaves, "depth": depth}


def _blocks(caps, b):
    return sum(-(-x // b) for x in caps)


def _chain(parent, x):
    out = []
    while x >= 0:
        out.append(x)
        x = parent[x]
    return out[::-1]


def _grow_forest(ctx, f):
    """Creates the forest's nodes; the pools already hold their rows."""
    parent, length, cap = f["parent"], f["len"], f["cap"]
    n = len(parent)
    i = 0
    done = 0  # nodes whose tokens are committed
    while i < n:
        p = parent[i]
        if p >= done:
            full = [k for k in range(done, i) if length[k]]
            ctx.kv_commit(np.array(full, np.int32), np.array([length[k] for k in full], np.int32))
            done = i
        if p < 0:
            ctx.new_root(cap[i])
            i += 1
            continue
        j = i + 1
        while j < n and parent[j] == p and cap[j] == cap[i]:
            j += 1
        ctx.fork(p, j - i, cap[i])
        i = j
    full = [k for k in range(done, n) if length[k]]
    if full:
        ctx.kv_commit(np.array(full, np.int32), np.array([length[k] for k in full], np.int32))


# ---- inputs -------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _normal(shape, g):
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEVICE)
    t.normal_(generator=g)
    return t


def _pool_blocks(c, caps, batches=1):
    # with 16-token blocks the library keeps the pool's last block free
    return _blocks(caps, c["block"]) * batches + (1 if c["block"] < 32 else 0)


def _pools(c, blocks, g):
    """K [Hkv][R][D] and V [Hkv][R / 16][D][16], random rows (g) or zeros."""
    rows = blocks * c["block"]
    k = torch.empty((c["hkv"], rows, c["d"]), dtype=torch.bfloat16, device=DEVICE)
    v = torch.empty((c["hkv"], rows // 16, c["d"], 16), dtype=torch.bfloat16, device=DEVICE)
    for t in (k, v):
        for h in range(c["hkv"]):
            t[h].zero_() if g is None else t[h].normal_(generator=g)
    return k, v


def _outputs(c, rows):
    out = torch.empty((rows, c["hq"], c["d"]), dtype=torch.float32, device=DEVICE)
    lse = torch.empty((rows, c["hq"]), dtype=torch.float32, device=DEVICE)
    return out, lse


def _bytes(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device=DEVICE)


def _scale(c):
    return 1.0 / math.sqrt(c["d"])


def _forest_inputs(c, seed):
    """Forest, pools and queries (and, for a step, the new tokens)."""
    f = _forest(c)
    g = _gen(seed)
    k, v = _pools(c, _pool_blocks(c, f["cap"]), g)
    n = len(f["leaves"])
    sets = STEP_SETS if c["kind"] == "step" else 1
    q = _normal((sets, n, c["hq"], c["d"]), g)
    new = _normal((sets, 2, n, c["hkv"], c["d"]), g) if c["kind"] == "step" else None
    return f, k, v, q, new


def _prefill_lens(c):
    r = random.Random(c["shape_seed"])
    return [r.randint(c["new_lo"], c["new_hi"]) for _ in range(c["rows"])]


def _rollout_lens(c):
    r = random.Random(c["shape_seed"])
    return [r.randint(c["new_lo"], c["new_hi"]) for _ in range(c["prompts"])]


def _rollout_caps(c, lens):
    caps = list(lens)
    for lv in range(c["levels"]):
        caps += [c["seg"]] * (c["prompts"] << (lv + 1))
    return caps


def _rollout_inputs(c, seed):
    lens = _rollout_lens(c)
    g = _gen(seed)
    n = sum(lens)
    prompt = (_normal((n, c["hq"], c["d"]), g), _normal((n, c["hkv"], c["d"]), g), _normal((n, c["hkv"], c["d"]), g))
    levels = []
    for lv in range(c["levels"]):
        w = c["prompts"] << (lv + 1)
        levels.append((_normal((c["seg"], w, c["hq"], c["d"]), g), _normal((c["seg"], 2, w, c["hkv"], c["d"]), g)))
    return lens, prompt, levels


class _State:
    pass


def prepare(case, seed):
    c = dict(case)
    s = _State()
    s.c, s.kind, s.scale = c, c["kind"], _scale(c)
    if s.kind in ("decode", "step"):
        s.f, s.k, s.v, q, new = _forest_inputs(c, seed)
        s.leaves = np.array(s.f["leaves"], np.int32)
        s.q = list(q)
        s.out, s.lse = _outputs(c, len(s.leaves))
        s.node_len = None
        if s.kind == "step":
            s.new = [(x[0], x[1]) for x in new]
            s.ones = np.ones(len(s.leaves), np.int32)
            s.node_len = torch.zeros(len(s.f["parent"]), dtype=torch.int32, device=DEVICE)
        _open_forest(s)
        s.ws = _bytes(s.ws_need)
    elif s.kind == "advantage":
        s.f = _forest(c)
        g = _gen(seed)
        s.leaves = np.array(s.f["leaves"], np.int32)
        s.rewards = (torch.rand(len(s.leaves), generator=g, device=DEVICE) < 0.5).float()
        s.adv = torch.empty(len(s.leaves), dtype=torch.float32, device=DEVICE)
        # the call reads the tree alone, so no keys and values are made
        blocks = _pool_blocks(c, s.f["cap"])
        elems = c["hkv"] * blocks * c["block"] * c["d"]
        s.k = torch.empty(elems, dtype=torch.bfloat16, device=DEVICE)
        s.v = torch.empty(elems, dtype=torch.bfloat16, device=DEVICE)
        s.ctx = Context(c["hq"], c["hkv"], c["d"], blocks, len(s.f["parent"]), s.k, s.v, c["block"])
        _grow_forest(s.ctx, s.f)
        s.ws = _bytes(s.ctx.advantage_workspace_size(s.leaves))
    elif s.kind == "prefill":
        lens = _prefill_lens(c)
        g = _gen(seed)
        n = sum(lens)
        s.q = _normal((n, c["hq"], c["d"]), g)
        s.knew, s.vnew = _normal((n, c["hkv"], c["d"]), g), _normal((n, c["hkv"], c["d"]), g)
        s.lens, s.ntok = lens, np.array(lens, np.int32)
        s.batch_blocks = _blocks(lens, c["block"])
        s.prefix_blocks = -(-c["prefix"] // c["block"])
        s.blocks = s.batch_blocks * BATCHES + s.prefix_blocks + (1 if c["block"] < 32 else 0)
        s.k, s.v = _pools(c, s.blocks, None)
        if c["prefix"]:
            rows = s.prefix_blocks * c["block"]
            s.k[:, :rows].normal_(generator=g)
            s.v[:, :rows // 16].normal_(generator=g)
        s.out, s.lse = _outputs(c, n)
        _open_prefill(s)
        nodes = _prefill_nodes(s)
        s.ws = _bytes(s.ctx.prefill_workspace_size(nodes, s.ntok))
        _open_prefill(s)
    else:
        s.lens, s.prompt, levels = _rollout_inputs(c, seed)
        s.ntok = np.array(s.lens, np.int32)
        s.levels = [([q[t] for t in range(c["seg"])], [(kv[t, 0], kv[t, 1]) for t in range(c["seg"])])
                    for q, kv in levels]
        caps = _rollout_caps(c, s.lens)
        s.per = len(caps)
        s.blocks = _pool_blocks(c, caps, BATCHES)
        s.k, s.v = _pools(c, s.blocks, None)
        s.node_len = torch.zeros(s.per * BATCHES, dtype=torch.int32, device=DEVICE)
        s.prompt_out = _outputs(c, sum(s.lens))
        s.outs, s.views = [], []
        for lv in range(c["levels"]):
            w = c["prompts"] << (lv + 1)
            o = torch.empty((c["seg"], w, c["hq"], c["d"]), dtype=torch.float32, device=DEVICE)
            l = torch.empty((c["seg"], w, c["hq"]), dtype=torch.float32, device=DEVICE)
            s.outs.append((o, l))
            s.views.append([(o[t], l[t]) for t in range(c["seg"])])
        s.ws = _bytes(64 << 20)
        _open_rollout(s)
    return s


def _open_forest(s):
    c = s.c
    s.ctx = Context(c["hq"], c["hkv"], c["d"], s.k.shape[1] // c["block"], len(s.f["parent"]), s.k, s.v, c["block"],
                    node_len=s.node_len)
    _grow_forest(s.ctx, s.f)
    s.ws_need = s.ctx.workspace_size(s.leaves)
    s.steps = 0


def _open_prefill(s):
    c = s.c
    s.ctx = Context(c["hq"], c["hkv"], c["d"], s.blocks, 1 + BATCHES * c["rows"], s.k, s.v, c["block"])
    s.used = 0
    if c["prefix"]:
        s.root = s.ctx.new_root(c["prefix"])
        s.ctx.kv_commit([s.root], [c["prefix"]])


def _prefill_nodes(s):
    if s.c["prefix"]:
        return np.array([s.ctx.fork(s.root, 1, n)[0] for n in s.lens], np.int32)
    return np.array([s.ctx.new_root(n) for n in s.lens], np.int32)


def _open_rollout(s):
    c = s.c
    s.ctx = Context(c["hq"], c["hkv"], c["d"], s.blocks, s.per * BATCHES, s.k, s.v, c["block"], node_len=s.node_len)
    s.used = 0


# ---- one pass -----------------------------------------------------------------


def run(state):
    return _RUN[state.kind](state)


def _run_decode(s):
    s.ctx.tree_decode(s.leaves, s.q[0], s.scale, s.out, s.lse, s.ws)
    return {"out": s.out, "lse": s.lse}


def _run_step(s):
    if s.steps == s.c["seg"]:
        _open_forest(s)
    i = s.steps % STEP_SETS
    s.ctx.kv_append(s.leaves, s.ones, s.new[i][0], s.new[i][1])
    s.ctx.tree_decode(s.leaves, s.q[i], s.scale, s.out, s.lse, s.ws)
    s.steps += 1
    return {"out": s.out, "lse": s.lse, "node_len": s.node_len}


def _run_prefill(s):
    if s.used == BATCHES:
        _open_prefill(s)
    nodes = _prefill_nodes(s)
    s.ctx.prefill(nodes, s.ntok, s.q, s.knew, s.vnew, s.scale, s.out, s.lse, s.ws)
    b0 = (s.prefix_blocks + s.used * s.batch_blocks) * s.c["block"]
    b1 = b0 + s.batch_blocks * s.c["block"]
    s.used += 1
    return {"out": s.out, "lse": s.lse, "k": s.k[:, b0:b1], "v": s.v[:, b0 // 16:b1 // 16]}


def _run_advantage(s):
    s.ctx.tree_advantage(s.leaves, s.rewards, s.adv, s.ws, s.c["weighting"])
    return {"adv": s.adv}


def _run_rollout(s):
    c = s.c
    if s.used == BATCHES:
        _open_rollout(s)
    ctx = s.ctx
    s.used += 1
    paths = np.array([ctx.new_root(n) for n in s.lens], np.int32)
    q, k, v = s.prompt
    need = ctx.prefill_workspace_size(paths, s.ntok)
    if need > s.ws.numel():
        s.ws = _bytes(need)
    ctx.prefill(paths, s.ntok, q, k, v, s.scale, s.prompt_out[0], s.prompt_out[1], s.ws)
    for lv in range(c["levels"]):
        paths = np.array([x for p in paths for x in ctx.fork(int(p), 2, c["seg"])], np.int32)
        ones = np.ones(len(paths), np.int32)
        qs, kvs = s.levels[lv]
        for t in range(c["seg"]):
            ctx.kv_append(paths, ones, kvs[t][0], kvs[t][1])
            if t == 0:
                need = ctx.workspace_size(paths)
                if need > s.ws.numel():
                    s.ws = _bytes(need)
            ctx.tree_decode(paths, qs[t], s.scale, s.views[lv][t][0], s.views[lv][t][1], s.ws)
    return {"prompt": s.prompt_out, "steps": s.outs}


_RUN = {"decode": _run_decode, "step": _run_step, "prefill": _run_prefill, "advantage": _run_advantage,
        "rollout": _run_rollout}


# ---- what a pass cannot do without ----------------------------------------------


def _depth_tokens(f, extra=0):
    tok = [0] * len(f["parent"])
    for i, p in enumerate(f["parent"]):
        tok[i] = f["len"][i] + (tok[p] if p >= 0 else 0)
    return sum(tok[x] + extra for x in f["leaves"])


def _on_chains(f):
    seen = set()
    for x in f["leaves"]:
        while x >= 0 and x not in seen:
            seen.add(x)
            x = f["parent"][x]
    return seen


def work(case):
    c = dict(case)
    kv, q, o = c["hkv"] * c["d"] * 4, c["hq"] * c["d"] * 2, c["hq"] * (c["d"] + 1) * 4
    fl = 4 * c["d"] * c["hq"]
    if c["kind"] in ("decode", "step"):
        f = _forest(c)
        n = len(f["leaves"])
        # a step at the middle of its segment: the new token's K and V are read and written
        half = c["seg"] // 2 if c["kind"] == "step" else 0
        unique = sum(f["len"][i] for i in _on_chains(f)) + n * half
        extra = 2 * n * kv if c["kind"] == "step" else 0
        return {"bytes": unique * kv + extra + n * (q + o), "flops": fl * _depth_tokens(f, half)}
    if c["kind"] == "prefill":
        lens = _prefill_lens(c)
        p = c["prefix"]
        return {"bytes": sum(lens) * (2 * kv + q + o) + p * kv,
                "flops": fl * sum(n * p + n * (n + 1) // 2 for n in lens)}
    if c["kind"] == "advantage":
        f = _forest(c)
        pairs = sum(f["depth"][x] for x in f["leaves"])
        return {"bytes": 12 * len(f["leaves"]) + 4 * len(f["parent"]), "flops": 8 * pairs}
    lens = _rollout_lens(c)
    b = sum(lens) * (2 * kv + q + o)
    w = fl * sum(n * (n + 1) // 2 for n in lens)
    for lv in range(c["levels"]):
        per = 2 << lv
        for t in range(1, c["seg"] + 1):
            done = sum((2 << j) * c["seg"] for j in range(lv))
            b += sum(n + done + per * t for n in lens) * kv + len(lens) * per * (2 * kv + q + o)
            w += fl * sum(per * (n + lv * c["seg"] + t) for n in lens)
    return {"bytes": b, "flops": w}


def tolerance(case):
    return _TOLERANCE[case["kind"]]


# About four times the error against 64 bits: 2e-6 with fp32 partial rows
# (two-term bf16 weights, fp32 sums), 8e-5 where a large decode keeps its
# partial rows in block floating point (2^-13 of a group's largest value).
_TOLERANCE = {
    "decode": {"rel": 3e-4, "max": 3e-3},
    "step": {"rel": 3e-4, "max": 3e-3},
    "prefill": {"rel": 8e-6, "max": 2e-4},
    "advantage": {"rel": 2e-7, "max": 1e-6},
    "rollout": {"rel": 3e-4, "max": 3e-3},
}


# ---- the same in 64 bits --------------------------------------------------------


def _attend(q, k, v, scale, mask=None):
    """q [Hkv, M, D], k and v [Hkv, L, D] in fp64: outputs [Hkv, M, D] and lse [Hkv, M]."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) * scale
    if mask is not None:
        s = s.masked_fill(mask, float("-inf"))
    lse = torch.logsumexp(s, dim=-1)
    return torch.matmul(torch.exp(s - lse.unsqueeze(-1)), v), lse


def _v_rows(v):
    """[Hkv][R / 16][D][16] -> [Hkv][R][D]"""
    h, n, d, w = v.shape
    return v.permute(0, 1, 3, 2).reshape(h, n * w, d)


def _exact_decode(c, seed):
    f, k, v, q, new = _forest_inputs(c, seed)
    n, hkv, hq, d = len(f["leaves"]), c["hkv"], c["hq"], c["d"]
    g = hq // hkv
    begin, at = [], 0
    for cp in f["cap"]:
        begin.append(at * c["block"])
        at += -(-cp // c["block"])
    out = torch.empty((n, hq, d), dtype=torch.float64, device=DEVICE)
    lse = torch.empty((n, hq), dtype=torch.float64, device=DEVICE)
    for i, x in enumerate(f["leaves"]):
        ks, vs = [], []
        for y in _chain(f["parent"], x):
            b, m = begin[y], f["len"][y]
            if m:
                ks.append(k[:, b:b + m].double())
                vs.append(_v_rows(v[:, b // 16:-(-(b + m) // 16)])[:, b % 16:b % 16 + m].double())
        if new is not None:
            ks.append(new[0, 0, i].double().unsqueeze(1))
            vs.append(new[0, 1, i].double().unsqueeze(1))
        o, l = _attend(q[0, i].double().view(hkv, g, d), torch.cat(ks, 1), torch.cat(vs, 1), _scale(c))
        out[i], lse[i] = o.reshape(hq, d), l.reshape(hq)
    r = {"out": out, "lse": lse}
    if new is not None:
        r["node_len"] = None
    return r


def _causal(c, q, k, v, pk, pv):
    """Rows of one sequence, [n, H, D] each, over a prefix pk / pv [Hkv, P, D] (or None)."""
    n, hkv, d = q.shape[0], c["hkv"], c["d"]
    g = c["hq"] // hkv
    kk, vv = k.permute(1, 0, 2).double(), v.permute(1, 0, 2).double()
    p = 0
    if pk is not None:
        p = pk.shape[1]
        kk, vv = torch.cat([pk, kk], 1), torch.cat([pv, vv], 1)
    qq = q.view(n, hkv, g, d).permute(1, 2, 0, 3).reshape(hkv, g * n, d).double()
    pos = torch.arange(n, device=DEVICE).repeat(g) + p
    mask = torch.arange(p + n, device=DEVICE).unsqueeze(0) > pos.unsqueeze(1)
    outs, lses = [], []
    for h in range(hkv):
        o, l = _attend(qq[h:h + 1], kk[h:h + 1], vv[h:h + 1], _scale(c), mask)
        outs.append(o), lses.append(l)
    o = torch.cat(outs).view(hkv, g, n, d).permute(2, 0, 1, 3).reshape(n, c["hq"], d)
    return o, torch.cat(lses).view(hkv, g, n).permute(2, 0, 1).reshape(n, c["hq"])


def _exact_prefill(c, seed):
    s = prepare(c, seed)
    rows = s.batch_blocks * c["block"]
    k = torch.zeros((c["hkv"], rows, c["d"]), dtype=torch.float64, device=DEVICE)
    v = torch.zeros_like(k)
    p = c["prefix"]
    pk = s.k[:, :p].double() if p else None
    pv = _v_rows(s.v[:, :-(-p // 16)])[:, :p].double() if p else None
    outs, lses, at, b = [], [], 0, 0
    for n in s.lens:
        q, kn, vn = s.q[at:at + n], s.knew[at:at + n], s.vnew[at:at + n]
        o, l = _causal(c, q, kn, vn, pk, pv)
        outs.append(o), lses.append(l)
        k[:, b:b + n], v[:, b:b + n] = kn.permute(1, 0, 2).double(), vn.permute(1, 0, 2).double()
        at += n
        b += -(-n // c["block"]) * c["block"]
    v = v.view(c["hkv"], rows // 16, 16, c["d"]).permute(0, 1, 3, 2)
    return {"out": torch.cat(outs), "lse": torch.cat(lses), "k": k, "v": v}


def _exact_advantage(c, seed):
    f = _forest(c)
    n = len(f["leaves"])
    rew = (torch.rand(n, generator=_gen(seed), device=DEVICE) < 0.5).double().cpu().numpy()
    chains = [_chain(f["parent"], x) for x in f["leaves"]]
    members = {}
    for i, ch in enumerate(chains):
        for x in ch:
            members.setdefault(x, []).append(i)
    mean = {x: rew[m].mean() for x, m in members.items()}
    pooled, every = np.zeros(n), []
    for i, ch in enumerate(chains):
        if np.all(rew[members[ch[0]]] == rew[i]) or len(ch) < 2:
            continue
        a = np.array([rew[i] - mean[x] for x in ch[:-1]])
        w = np.array([len(members[x]) for x in ch[:-1]], float) if c["weighting"] else np.ones(len(a))
        pooled[i] = (w * a).sum() / w.sum()
        every.append(a)
    sigma = np.concatenate(every).std() if every else 0.0
    return {"adv": torch.from_numpy(pooled / sigma if sigma > 0 else pooled * 0)}


def _exact_rollout(c, seed):
    lens, (q, k, v), levels = _rollout_inputs(c, seed)
    hkv, g, d = c["hkv"], c["hq"] // c["hkv"], c["d"]
    outs, lses, paths, at = [], [], [], 0
    for n in lens:
        o, l = _causal(c, q[at:at + n], k[at:at + n], v[at:at + n], None, None)
        outs.append(o), lses.append(l)
        paths.append((k[at:at + n].permute(1, 0, 2).double(), v[at:at + n].permute(1, 0, 2).double()))
        at += n
    steps = []
    for lq, kv in levels:
        paths = [p for p in paths for _ in range(2)]
        o = torch.empty((c["seg"], len(paths), c["hq"], d), dtype=torch.float64, device=DEVICE)
        l = torch.empty((c["seg"], len(paths), c["hq"]), dtype=torch.float64, device=DEVICE)
        for i, (pk, pv) in enumerate(paths):
            for t in range(c["seg"]):
                pk = torch.cat([pk, kv[t, 0, i].double().unsqueeze(1)], 1)
                pv = torch.cat([pv, kv[t, 1, i].double().unsqueeze(1)], 1)
                a, b = _attend(lq[t, i].double().view(hkv, g, d), pk, pv, _scale(c))
                o[t, i], l[t, i] = a.reshape(c["hq"], d), b.reshape(c["hq"])
            paths[i] = (pk, pv)
        steps.append((o, l))
    return {"prompt": (torch.cat(outs), torch.cat(lses)), "steps": steps}


def exact(case, seed):
    c = dict(case)
    return {"decode": _exact_decode, "step": _exact_decode, "prefill": _exact_prefill,
            "advantage": _exact_advantage, "rollout": _exact_rollout}[c["kind"]](c, seed)
