"""The workloads whose speed this library is held to: what they are, how their inputs are made, and how one pass runs.

Three kinds of work, each through the entry points of ``paper_2605_07230_amd.binding`` as a serving program calls them:

``step``     one tree-verification step: tree attention, LM-head projection with guidance, top-k and softmax
             statistics, relaxed acceptance, path selection (the four calls of a decode iteration)
``commit``   the copy of the accepted path's keys and values into the prefix cache of every decoder layer
``weights``  the drafter-training weight mask over whole target-generated sequences

Sizes are the repository's own configurations (``workloads.make_config``, ``bench.py``, the GPU tests) and the ranges
between them.  Inputs follow the laws of ``workloads.py`` but are drawn on the GPU, from the seed alone.
"""
from __future__ import annotations

import random

import numpy as np
import torch

from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

STEP = dict(kind="step", dtype="bf16", prompts=1, guidance=True, heads=32, kv_heads=32, head_dim=128, hidden=4096, vocab=16384,
            prefix_min=312, prefix_max=312, nodes_min=60, nodes_max=60, depth_min=6, depth_max=6, cfg_scale=5.0, top_k=2000,
            tau_pos=0.85, tau_seq=0.5, cfg_mix="hidden", packed=True, features="hidden", walk="sequential", shape_seed=0)


def listed():
    def step(name, **kw):
        return dict(STEP, name=name, **kw)

    return [
        # the smallest call: the fp32 configuration, one short unguided sequence; all launch and round-trip latency
        step("tiny_f32", dtype="f32", guidance=False, heads=8, kv_heads=8, head_dim=64, hidden=512, vocab=4096, prefix_min=256,
             prefix_max=256, nodes_min=15, nodes_max=15, depth_min=3, depth_max=3, cfg_scale=1.0, top_k=0, tau_pos=0.9,
             tau_seq=0.9, packed=False, cfg_mix="logits"),
        # one interactive user, 576-token image, 60-node tree: the step whose latency is felt
        step("janus"),
        # the same with the arguments' defaults: weights as the checkpoint holds them, guidance mixed on the logits
        step("janus_defaults", packed=False, cfg_mix="logits"),
        # one user, ~2400-token image, four times the vocabulary: the weight matrix streams
        step("lumina", vocab=65536, prefix_min=1289, prefix_max=1289, cfg_scale=3.0, tau_pos=0.95, tau_seq=0.925),
        # eight users at different points of their images with trees of different sizes
        step("batched", prompts=8, prefix_min=100, prefix_max=600, nodes_min=40, nodes_max=80, depth_min=4, depth_max=7, shape_seed=1),
        # a grouped-head model of another width with odd tree sizes, guidance on the logits, the longest-path walk
        step("grouped_ragged", prompts=5, kv_heads=8, hidden=2048, vocab=33088, prefix_min=90, prefix_max=1500, nodes_min=17,
             nodes_max=119, depth_min=3, depth_max=9, cfg_scale=3.0, cfg_mix="logits", walk="longest", shape_seed=2),
        # the benchmark's headline: four users, 1024-pixel image, 256-node trees
        step("stress", prompts=4, vocab=65536, prefix_min=4200, prefix_max=4200, nodes_min=256, nodes_max=256, depth_min=10,
             depth_max=10, cfg_scale=3.0, tau_pos=0.9, tau_seq=0.9, shape_seed=3),
        # one user at the same point: few (row, head) pairs, long prefix, large tree
        step("stress_one_user", vocab=65536, prefix_min=4200, prefix_max=4200, nodes_min=256, nodes_max=256, depth_min=10,
             depth_max=10, cfg_scale=3.0, tau_pos=0.9, tau_seq=0.9, shape_seed=4),
        # full drafter distributions: every rejection re-normalises the residual
        step("residual_walk", prompts=4, prefix_min=100, prefix_max=600, nodes_min=40, nodes_max=80, depth_min=4, depth_max=7,
             walk="residual", shape_seed=5),
        # similarity measured on the logits rows instead of the hidden states; guidance stretches what two rows do not share,
        # so near-duplicates sit near a cosine of 0.2 there and strangers near 0
        step("logit_space", prompts=2, prefix_min=200, prefix_max=500, nodes_min=40, nodes_max=80, depth_min=4, depth_max=7,
             features="logits", tau_pos=0.1, tau_seq=0.1, shape_seed=6),
        # the commit that follows every step: 30 decoder layers, eight users
        dict(name="commit", kind="commit", dtype="bf16", layers=30, prompts=8, guidance=True, kv_heads=32, head_dim=128, prefix_min=100,
             prefix_max=600, nodes_min=40, nodes_max=80, depth_min=4, depth_max=7, shape_seed=7),
        # the training mask over eight ~2400-token images
        dict(name="weights", kind="weights", dtype="bf16", seqs=8, seq_len=2356, hidden=4096),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _shape_fields(rng, most_nodes, most_prefix, prompts):
    """Prefix, tree-size and depth ranges of a batch: ragged half of the time."""
    ragged = prompts > 1 and rng.random() < 0.5
    nmax, pmax = _log_int(rng, 15, most_nodes), _log_int(rng, 24, most_prefix)
    dmax = rng.randint(3, min(10, nmax - 2))
    # a tree of n nodes holds one chain of its depth and at most ten children per node (three levels hold over a thousand)
    nmin = max(dmax + 2, nmax // 3) if ragged else nmax
    return dict(prefix_min=max(1, pmax // 6) if ragged else pmax, prefix_max=pmax, nodes_min=nmin, nodes_max=max(nmin, nmax),
                depth_min=max(3, dmax - 3) if ragged else dmax, depth_max=dmax, shape_seed=rng.randrange(1 << 20))


def draw(rng):
    """One more case of the ranges above, costing no more than ``stress``."""
    kind = rng.choices(["step", "commit", "weights"], [10, 1, 1])[0]
    if kind == "weights":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        hidden = 64 * rng.randint(4, 64)
        return dict(kind="weights", dtype=dtype, seqs=_log_int(rng, 1, 8), seq_len=_log_int(rng, 200, 2400), hidden=hidden)
    if kind == "commit":
        prompts = _log_int(rng, 1, 8)
        return dict(kind="commit", dtype="bf16", layers=rng.randint(12, 32), prompts=prompts, guidance=rng.random() < 0.8,
                    kv_heads=rng.choice([8, 32]), head_dim=rng.choice([64, 128]), **_shape_fields(rng, 128, 1300, prompts))
    top = listed()[6]
    while True:
        prompts = _log_int(rng, 1, 8)
        c = dict(STEP, prompts=prompts, guidance=rng.random() < 0.85, cfg_scale=rng.choice([3.0, 5.0]),
                 walk=rng.choice(["sequential", "sequential", "sequential", "longest", "residual"]),
                 features=rng.choice(["hidden"] * 5 + ["logits"]))
        if rng.random() < 0.1:
            # fp32: the small configuration's neighbourhood
            c.update(dtype="f32", packed=False, cfg_mix="logits", heads=8, kv_heads=rng.choice([2, 8]), head_dim=rng.choice([32, 64]),
                     hidden=rng.randint(64, 512), vocab=4 * rng.randint(200, 1024), top_k=rng.choice([0, 50]), tau_pos=0.9, tau_seq=0.9,
                     **_shape_fields(rng, 64, 320, prompts))
            return c
        c.update(kv_heads=rng.choice([32, 32, 32, 8]), head_dim=rng.choice([128, 128, 128, 64]),
                 hidden=rng.choice([4096, 4096, 4096, 2048, 128 * rng.randint(8, 40)]),
                 vocab=rng.choice([16384, 65536, 64 * rng.randint(64, 1024)]), top_k=rng.choice([2000, 2000, 2000, 0]),
                 packed=rng.random() < 0.8, **_shape_fields(rng, 256, 4200, prompts))
        c["cfg_mix"] = rng.choice(["hidden", "hidden", "hidden", "logits"]) if c["packed"] else "logits"
        if c["features"] == "logits":
            c.update(tau_pos=0.1, tau_seq=0.1)
        w, most = work(c), work(top)
        nodes = c["nodes_max"] * prompts
        if w["flops"] > most["flops"] / 2 or w["bytes"] > most["bytes"] or (not c["packed"] and nodes > 128) or nodes > 1024:
            continue
        # cosines of logits rows and residual rows are read at vocabulary width for every node
        if (c["features"] == "logits" or c["walk"] == "residual") and nodes * c["vocab"] > 400 * 16384:
            continue
        return c


# ------------------------------------------------------------------------------------------------ shapes of a case

def _rows(c):
    return c["prompts"] * (2 if c["guidance"] else 1)


def _shapes(c):
    """(prefix lengths per prompt, node counts per prompt, depths per prompt): functions of the case, not of the seed."""
    r = random.Random(c["shape_seed"])
    prefix = [r.randint(c["prefix_min"], c["prefix_max"]) for _ in range(c["prompts"])]
    nodes = [r.randint(c["nodes_min"], c["nodes_max"]) for _ in range(c["prompts"])]
    depth = [min(r.randint(c["depth_min"], c["depth_max"]), n - 1) for n in nodes]
    if c["prompts"] > 1:   # the ends of the ranges are part of the case
        prefix[0], prefix[-1] = c["prefix_max"], c["prefix_min"]
        nodes[0], nodes[-1] = c["nodes_max"], c["nodes_min"]
        depth = [min(d, n - 1) for d, n in zip(depth, nodes)]
    return prefix, nodes, depth


def _accepted(c):
    """Accepted tokens per prompt of a commit case."""
    r = random.Random(c["shape_seed"] + 1)
    return [r.randint(0, d) for d in _shapes(c)[2]]


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "weights":
        return {"bytes": c["seqs"] * c["seq_len"] * (c["hidden"] * e + 8), "flops": 4 * c["seqs"] * c["seq_len"] * c["hidden"]}
    per_prompt = 2 if c["guidance"] else 1
    if c["kind"] == "commit":
        tokens = sum(1 + n for n in _accepted(c)) * per_prompt
        return {"bytes": tokens * c["layers"] * c["kv_heads"] * c["head_dim"] * e * 2 * 2, "flops": 0}
    prefix, nodes, depth = _shapes(c)
    D, hq, hkv, h, V, N = c["head_dim"], c["heads"], c["kv_heads"], c["hidden"], c["vocab"], sum(nodes)
    nbytes = flops = 0
    for P, T, d in zip(prefix, nodes, depth):
        nbytes += per_prompt * ((P + T) * hkv * D * 2 * e + T * hq * (D * 2 * e + 4))   # keys, values, queries, outputs, lse
        flops += per_prompt * 4 * T * hq * D * (P + 1 + d // 2)
    nbytes += V * h * e + N * per_prompt * h * e + N * V * 4 + N * (12 + 24 + 16)       # weights, hidden rows, logits, scalars
    # guidance on the hidden rows is one product over N rows, on the logits two
    flops += 2 * h * V * N * (2 if c["guidance"] and c["cfg_mix"] == "logits" else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "commit":
        return "exact"
    # Against the same path in float64: fp32 results are off by at most 6e-7 (2-norm) and 2.5e-6 (largest); sums of
    # another order move the third of those digits.  bf16 attention, whose probabilities and outputs are rounded once
    # each, is off by 2.1e-3 and 1.7e-2, and dominates: logits are float32 sums of exact products.
    if case["kind"] == "weights" or case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    return {"rel": 8e-3, "max": 0.07}


# ------------------------------------------------------------------------------------------------ inputs

DEV = "cuda:0"


def _tree_arrays(c, rng):
    _, nodes, depth = _shapes(c)
    trees = [wl.grow_tree(rng, n, d) for n, d in zip(nodes, depth)]
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    return trees, off


def _zipf(vocab):
    pmf = np.arange(1, vocab + 1, dtype=np.float64) ** -1.1
    return pmf / pmf.sum()


def _tokens(trees, vocab, rng):
    """Drafted tokens: Zipf(1.1) over a permutation of the vocabulary, distinct among siblings, and their drafter probability."""
    pmf = _zipf(vocab)
    cum, perm = np.cumsum(pmf), rng.permutation(vocab).astype(np.int32)
    token, prob = [], []
    for t in trees:
        tok, pr = np.empty(len(t), np.int32), np.ones(len(t), np.float32)
        tok[0] = rng.integers(0, vocab)
        taken = {}
        for i in range(1, len(t)):
            mine = taken.setdefault(int(t[i]), set())
            while True:
                k = min(int(np.searchsorted(cum, rng.random(), side="right")), vocab - 1)
                if k not in mine:
                    break
            mine.add(k)
            tok[i], pr[i] = perm[k], pmf[k]
        token.append(tok)
        prob.append(pr)
    return np.concatenate(token), np.concatenate(prob)


def _hidden_rows(c, trees, off, token, w, gen, rng):
    """Target hidden states: near-duplicates of a parent or an earlier sibling as image regions give them, nudged towards
    the drafted children's LM-head rows as a trained drafter's proposals are; unconditional rows beside them."""
    N, h = int(off[-1]), c["hidden"]
    sigmas = (0.62, 0.43, 0.25, 0.14) if c["tau_pos"] == 0.9 else (0.1, 0.2, 0.25)
    x = torch.randn(N, h, device=DEV, generator=gen)
    parents, kids = [], []
    for t, lo in zip(trees, off[:-1].tolist()):
        sib = {}
        for i in range(len(t)):
            if i > 0:
                p, mine, r = int(t[i]), sib.setdefault(int(t[i]), []), rng.random()
                base = p if r < 0.2 else (mine[int(rng.integers(0, len(mine)))] if r < 0.5 and mine else -1)
                if base >= 0:
                    x[lo + i].mul_(float(sigmas[int(rng.integers(0, len(sigmas)))])).add_(x[lo + base])
                mine.append(i)
                parents.append(lo + p)
                kids.append(lo + i)
    hu = x + 0.5 * torch.randn(N, h, device=DEV, generator=gen) if c["guidance"] else None
    if kids:
        gain = torch.from_numpy(1.5 * rng.uniform(0.4, 1.6, len(kids)).astype(np.float32)).to(DEV)
        rows = w[torch.from_numpy(token[kids].astype(np.int64)).to(DEV)].float() * (gain / (0.02 * 0.02 * h))[:, None]
        # one pass per rank among siblings: no parent occurs twice in an addition, so the sums keep one order
        order, rank = {}, []
        for p in parents:
            order[p] = order.get(p, -1) + 1
            rank.append(order[p])
        rank = np.asarray(rank)
        for k in range(int(rank.max()) + 1):
            at = torch.from_numpy(np.nonzero(rank == k)[0]).to(DEV)
            x[torch.tensor(parents, device=DEV)[at]] += rows[at]
    return x, hu


def _draft_rows(c, trees, off, token, gen):
    """Full drafter distributions: siblings share a row, a Zipf(1.1) law over a random order of the vocabulary with 0.4 of
    the mass on the drafted tokens themselves."""
    N, V = int(off[-1]), c["vocab"]
    pmf = torch.from_numpy(_zipf(V).astype(np.float32)).to(DEV)
    out = torch.full((N, V), 1.0 / V, device=DEV)
    for t, lo in zip(trees, off[:-1].tolist()):
        for p in sorted(set(t[1:].tolist())):
            kids = np.nonzero(t == p)[0]
            row = 0.6 * pmf[torch.randperm(V, device=DEV, generator=gen)]
            wts = np.arange(1, len(kids) + 1) ** -1.1
            row[torch.from_numpy(token[lo + kids].astype(np.int64)).to(DEV)] += torch.from_numpy((0.4 * wts / wts.sum()).astype(np.float32)).to(DEV)
            out[torch.from_numpy(lo + kids).to(DEV)] = row
    return out


def _up(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _prepare_step(c, gen, rng):
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    prefix, nodes, _ = _shapes(c)
    trees, off = _tree_arrays(c, rng)
    per = 2 if c["guidance"] else 1
    S, N, B, V, h = _rows(c), int(off[-1]), c["prompts"], c["vocab"], c["hidden"]
    Na, Hq, Hkv, D = N * per, c["heads"], c["kv_heads"], c["head_dim"]
    row_trees = [t for t in trees for _ in range(per)]
    row_off = np.concatenate([[0], np.cumsum([len(t) for t in row_trees])]).astype(np.int32)
    depth = max(int(wl.node_depths(t).max()) for t in trees)

    def normal(*shape):
        return torch.randn(*shape, device=DEV, generator=gen).to(dt)

    w = (0.02 * torch.randn(V, h, device=DEV, generator=gen)).to(dt)
    token, prob = _tokens(trees, V, rng)
    hc, hu = _hidden_rows(c, trees, off, token, w, gen, rng)
    plen = [p for p in prefix for _ in range(per)]
    cap = max(plen)
    ctx = binding.Context(max_rows=S, max_nodes_total=Na, max_nodes_per_tree=max(nodes), max_prefix=cap, n_heads=Hq, head_dim=D, hidden=h, vocab=V)

    def f32(*n):
        return torch.empty(*n, dtype=torch.float32, device=DEV)

    def i32(*n):
        return torch.empty(*n, dtype=torch.int32, device=DEV)

    tree = dict(node_off=_up(off), parent=_up(np.concatenate(trees)), token=_up(token))
    scal = dict(q_tok=f32(N), m_int=f32(N), m_conv=f32(N), n_int=i32(N), n_conv=i32(N))
    rows = dict(logits=f32(N, V), row_thr=f32(N), row_lse=f32(N))
    hc, row_max = hc.to(dt), f32(N)
    attn = dict(node_off=_up(row_off), parent=_up(np.concatenate(row_trees)), prefix_len=_up(np.asarray(plen, np.int32)), q=normal(Na, Hq, D),
                k_tree=normal(Na, Hkv, D), v_tree=normal(Na, Hkv, D), k_cache=normal(S, Hkv, cap, D), v_cache=normal(S, Hkv, cap, D),
                out=torch.empty(Na, Hq, D, dtype=dt, device=DEV), lse=f32(Na, Hq), max_nodes_per_tree=max(nodes), max_prefix_len=cap)
    lm = dict(h_cond=hc, h_uncond=None if hu is None else hu.to(dt), w=binding.cascade_pack_lmhead_w(ctx, w) if c["packed"] else w,
              w_layout=binding.W_PACKED32 if c["packed"] else binding.W_ROWMAJOR, cfg_scale=c["cfg_scale"], temperature=1.0, top_k=c["top_k"],
              cfg_mix=binding.CFG_MIX_HIDDEN if c["cfg_mix"] == "hidden" else binding.CFG_MIX_LOGITS, row_max=row_max, **rows)
    acc = dict(tree, h_cond=hc, tau_pos=c["tau_pos"], tau_seq=c["tau_seq"], cos_parent=f32(N),
               feature_space=binding.FEATURES_LOGITS if c["features"] == "logits" else binding.FEATURES_HIDDEN, **rows, **scal)
    u = rng.integers(0, 1 << 24, N + B).astype(np.float32) / np.float32(1 << 24)
    sel = dict(tree, draft_prob=_up(prob), u=_up(u[:N]), u_bonus=_up(u[N:]), eps_tvd=0.5, max_depth=depth,
               mode=binding.WALK_LONGEST if c["walk"] == "longest" else binding.WALK_SEQUENTIAL, accept_len=i32(B), path_nodes=i32(B, depth),
               emitted=i32(B, depth + 1), terminal=i32(B), tvd_used=f32(B),
               draft_dist=_draft_rows(c, trees, off, token, gen) if c["walk"] == "residual" else None, **rows, **scal)
    outputs = dict(rows, **scal, attn_out=attn["out"], attn_lse=attn["lse"], row_max=row_max, cos_parent=acc["cos_parent"],
                   **{k: sel[k] for k in ("accept_len", "path_nodes", "emitted", "terminal", "tvd_used")})
    return dict(kind="step", ctx=ctx, attn=attn, lm=lm, acc=acc, sel=sel, outputs=outputs)


def _prepare_commit(c, gen, rng):
    prefix, nodes, _ = _shapes(c)
    trees, off = _tree_arrays(c, rng)
    per = 2 if c["guidance"] else 1
    S, B, L, Hkv, D = _rows(c), c["prompts"], c["layers"], c["kv_heads"], c["head_dim"]
    row_off = np.concatenate([[0], np.cumsum([n for n in nodes for _ in range(per)])]).astype(np.int32)
    n_acc, depth = _accepted(c), max(int(wl.node_depths(t).max()) for t in trees)
    path = -np.ones((B, depth), np.int32)
    for b, t in enumerate(trees):   # a random node of the accepted depth, and the way down to it
        d = wl.node_depths(t)
        x = int(rng.choice(np.nonzero(d == n_acc[b])[0]))
        for j in range(n_acc[b] - 1, -1, -1):
            path[b, j], x = x, int(t[x])
    plen = np.asarray([p for p in prefix for _ in range(per)], np.int32)
    cap = -(-(int(plen.max()) + depth + 4) // 8) * 8
    ctx = binding.Context(max_rows=S, max_nodes_total=int(row_off[-1]), max_nodes_per_tree=max(nodes), max_prefix=cap, n_heads=Hkv, head_dim=D,
                          hidden=128, vocab=64)

    def normal(*shape):
        return torch.empty(*shape, dtype=torch.bfloat16, device=DEV).normal_(generator=gen)

    kc = normal(L, S, Hkv, cap, D)
    vc = normal(L, S, Hkv, cap, D)
    args = dict(node_off=_up(row_off), row_prompt=_up((np.arange(S) // per).astype(np.int32)), accept_len=_up(np.asarray(n_acc, np.int32)),
                path_nodes=_up(path), k_tree=normal(L, int(row_off[-1]), Hkv, D), v_tree=normal(L, int(row_off[-1]), Hkv, D), k_cache=kc, v_cache=vc,
                prefix_len=_up(plen), prefix_len_out=torch.empty(S, dtype=torch.int32, device=DEV))
    return dict(kind="commit", ctx=ctx, args=args, outputs=dict(k_cache=kc, v_cache=vc, prefix_len_out=args["prefix_len_out"]))


def _prepare_weights(c, gen, rng):
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    B, K, h = c["seqs"], c["seq_len"], c["hidden"]
    x = torch.randn(B, K, h, device=DEV, generator=gen)
    # uniform regions and boundaries: a position keeps its predecessor's feature plus noise, or starts afresh
    sigma = torch.from_numpy(np.where(rng.random((B, K)) < 0.6, rng.choice([0.1, 0.2, 0.3, 0.6], (B, K)), 0.0).astype(np.float32)).to(DEV)
    keep = (sigma > 0).to(torch.float32)
    noise = torch.where(sigma > 0, sigma, torch.ones_like(sigma))
    for k in range(1, K):
        x[:, k] = keep[:, k, None] * x[:, k - 1] + noise[:, k, None] * x[:, k]
    ctx = binding.Context(max_rows=1, max_nodes_total=1, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=64, vocab=64)
    args = dict(features=x.to(dt).contiguous(), tau_seq=0.9, c=2.0, weights=torch.empty(B, K, device=DEV), cos_next=torch.empty(B, K, device=DEV))
    return dict(kind="weights", ctx=ctx, args=args, outputs=dict(weights=args["weights"], cos_next=args["cos_next"]))


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    return {"step": _prepare_step, "commit": _prepare_commit, "weights": _prepare_weights}[case["kind"]](case, gen, rng)


# ------------------------------------------------------------------------------------------------ one pass

def run(state):
    ctx = state["ctx"]
    if state["kind"] == "step":
        binding.tree_verify_attn(ctx, **state["attn"])
        binding.lmhead_softmax_cfg(ctx, **state["lm"])
        binding.cascade_accept(ctx, **state["acc"])
        binding.select_path(ctx, **state["sel"])
    elif state["kind"] == "commit":
        binding.kv_commit(ctx, **state["args"])
    else:
        binding.convergence_weights(ctx, **state["args"])
    return state["outputs"]
