"""What users of this library have it do, as a list of measurable cases.

A case is one rollout tree, one head configuration and one way of calling the
library.  Trees are the shapes of the benchmark (a prompt with sampled answers, a
multi-turn agent forest, a deep tree, a mixed forest of short segments), inputs
are i.i.d. N(0,1) as there.  The ways of calling:

  train     attention of one layer of a training step on a tree that the program
            keeps for all its layers: forward, then backward
  step      the same for a batch that has just arrived: the tree is built,
            scheduled and uploaded inside the pass (one step of bench.py)
  forward   scoring: forward only, on a kept tree
  pushpop   an executor that holds one root path at a time: a forward call when a
            segment is pushed, a backward call when it is popped
  leaforder the same work in the order of dta_tree_plan, long pops cut in chunks
"""
import math

import numpy as np
import torch

import paper_2602_00482_amd as dta

BF16, F32 = "bf16", "f32"


def _case(name, call, heads, dtype, **tree):
    q_heads, kv_heads, head_dim = heads
    return dict(name=name, call=call, q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, dtype=dtype, **tree)


def listed():
    return [
        # smallest: the 384-token fp32 tree that accuracy checks and unit tests of a trainer run
        _case("tiny_tree_f32", "train", (4, 4, 64), F32, shape="fan", prompt=128, fan="4x32 2x16"),
        # fp32 in earnest: a group of short answers trained or checked without bf16 rounding
        _case("answer_group_f32", "train", (32, 8, 128), F32, shape="prompts", roots=1, prompt_lo=256, prompt_hi=256,
              answers=16, answer_lo=64, answer_hi=512, tree_seed=1002),
        # a group of short answers (about 2.5K tokens): few tiles, latency and launches count
        _case("short_group", "train", (32, 8, 128), BF16, shape="prompts", roots=1, prompt_lo=128, prompt_hi=128,
              answers=16, answer_lo=32, answer_hi=256, tree_seed=1002),
        # one prompt with 16 answers of up to 2K tokens, arriving as a new batch
        _case("answer_group", "step", (32, 8, 128), BF16, shape="prompts", roots=1, prompt_lo=1024, prompt_hi=1024,
              answers=16, answer_lo=256, answer_hi=2048, tree_seed=1002),
        # multi-turn agent rollouts under one system prompt
        _case("agent_forest", "train", (32, 8, 128), BF16, shape="agents", prompt=4096, dialogues=8, turns=6,
              turn_lo=128, turn_hi=1024, tree_seed=1003),
        # the same rollouts in a model with head_dim 64
        _case("agent_forest_d64", "train", (32, 8, 64), BF16, shape="agents", prompt=4096, dialogues=8, turns=6,
              turn_lo=128, turn_hi=1024, tree_seed=1003),
        # largest: deep long-context tree, 277 504 tokens, every rollout 20 480 long
        _case("deep_tree", "step", (32, 8, 128), BF16, shape="fan", prompt=16384,
              fan="2x512 2x512 2x512 2x512 2x512 2x512 2x512 2x512"),
        # many trees of short segments, 64 query heads
        _case("mixed_forest", "step", (64, 8, 128), BF16, shape="mixed", roots=64, tokens=262144, tree_seed=1005),
        # little to share: 8 short questions with 8 answers each, scored by a reference model
        _case("score_answers", "forward", (32, 8, 128), BF16, shape="prompts", roots=8, prompt_lo=100, prompt_hi=240,
              answers=8, answer_lo=800, answer_hi=2500, tree_seed=1007),
        # plain multi-head attention (no grouped heads) over ragged two-answer pairs, as in preference training
        _case("answer_pairs_mha", "train", (16, 16, 128), BF16, shape="prompts", roots=16, prompt_lo=700,
              prompt_hi=1100, answers=2, answer_lo=400, answer_hi=1000, tree_seed=1006),
        # executors bounded by the longest path: one call per segment and direction
        _case("push_pop_group", "pushpop", (32, 8, 128), BF16, shape="prompts", roots=1, prompt_lo=1024,
              prompt_hi=1024, answers=16, answer_lo=256, answer_hi=2048, tree_seed=1002),
        # ... and the leaf-order plan over a forest of short segments: hundreds of small calls
        _case("leaf_order_forest", "leaforder", (64, 8, 128), BF16, shape="mixed", roots=8, tokens=16384, block=2048,
              tree_seed=1005),
    ]


def draw(rng):
    """One more case of the same ranges: any shape, head configuration and way of
    calling, sizes log-uniform between the tiny tree and (within the work bounds
    below) the deep tree."""

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        call = rng.choice(["train", "train", "train", "step", "step", "forward", "pushpop", "leaforder"])
        dtype = rng.choice([BF16, BF16, BF16, F32])
        heads = rng.choice([(32, 8), (32, 8), (64, 8), (16, 16), (8, 2), (16, 2), (4, 4), (12, 4), (16, 1)])
        d = rng.choice([128, 128, 64])
        shape = rng.choice(["prompts", "agents", "fan", "mixed"])
        if shape == "prompts":
            lo = log_int(16, 1024)
            plo = log_int(32, 2048)
            tree = dict(roots=log_int(1, 32), prompt_lo=plo, prompt_hi=2 * plo, answers=rng.randint(2, 16),
                        answer_lo=lo, answer_hi=lo * rng.randint(2, 8))
        elif shape == "agents":
            lo = log_int(16, 256)
            tree = dict(prompt=log_int(64, 4096), dialogues=rng.randint(2, 8), turns=rng.randint(2, 6), turn_lo=lo,
                        turn_hi=lo * rng.randint(2, 8))
        elif shape == "fan":
            levels = rng.randint(1, 6)
            tree = dict(prompt=log_int(64, 16384),
                        fan=" ".join("%dx%d" % (rng.randint(2, 3), log_int(16, 512)) for _ in range(levels)))
        else:
            tree = dict(roots=rng.randint(2, 64), tokens=log_int(1024, 262144))
        if call == "leaforder":
            tree["block"] = rng.choice([256, 1024, 2048])
        case = _case("", call, heads + (d,), dtype, shape=shape, tree_seed=rng.randint(1, 1 << 30), **tree)
        del case["name"]
        parent, seg = _tree(case)
        pairs = _pairs(parent, seg)
        flops = pairs * case["q_heads"] * d * (4 if call == "forward" else 14)
        # the tiny tree's size at least; fp32 up to some 30K-token batches, executors up to a thousand segments
        most = 1e12 if dtype == F32 else 3e13 if call in ("pushpop", "leaforder") else 1e14
        if int(seg.sum()) >= 256 and flops <= most and (call not in ("pushpop", "leaforder") or len(seg) <= 600):
            return case


# ---- trees: parent[] / seg_len[] -------------------------------------------------

def _tree(case):
    rng = np.random.default_rng(case.get("tree_seed", 0))
    parent, seg = [], []

    def node(up, length):
        parent.append(up)
        seg.append(int(length))
        return len(parent) - 1

    shape = case["shape"]
    if shape == "prompts":          # roots x (prompt, answers)
        for _ in range(case["roots"]):
            root = node(-1, rng.integers(case["prompt_lo"], case["prompt_hi"] + 1))
            for n in rng.integers(case["answer_lo"], case["answer_hi"] + 1, size=case["answers"]):
                node(root, n)
    elif shape == "agents":         # system prompt, dialogues whose turns branch with probability 0.3
        root = node(-1, case["prompt"])
        for _ in range(case["dialogues"]):
            tips = [root]
            for turn in range(case["turns"]):
                tips = [node(tip, rng.integers(case["turn_lo"], case["turn_hi"] + 1))
                        for tip in tips for _ in range(2 if turn and rng.random() < 0.3 else 1)]
    elif shape == "fan":            # every node of a level has the same number of equal children
        tips = [node(-1, case["prompt"])]
        for level in case["fan"].split():
            kids, length = (int(x) for x in level.split("x"))
            tips = [node(tip, length) for tip in tips for _ in range(kids)]
    else:                           # "mixed": trees of random depth and branching, segments log-uniform,
        lengths = []                # all lengths scaled together to the token count
        for _ in range(case["roots"]):
            tips = [node(-1, 0)]
            lengths.append(rng.uniform(512, 8192))
            for _ in range(rng.integers(1, 6)):
                nxt = []
                for tip in tips:
                    for _ in range(rng.integers(1, 5)):
                        nxt.append(node(tip, 0))
                        lengths.append(math.exp(rng.uniform(math.log(32), math.log(2048))))
                tips = nxt
        scale = min(1.0, case["tokens"] / sum(lengths))
        seg = [max(8, round(n * scale)) for n in lengths]
    return np.asarray(parent, dtype=np.int32), np.asarray(seg, dtype=np.int32)


def _pairs(parent, seg):
    """(query, visible key) pairs; parents come before their children here."""
    depth = np.zeros(len(seg), dtype=np.int64)
    for u, p in enumerate(parent):
        if p >= 0:
            depth[u] = depth[p] + seg[p]
    n = seg.astype(np.int64)
    return int((n * depth + n * (n + 1) // 2).sum())


def _push_pop_calls(tree, parent, seg):
    """(is_backward, first row, end row) in the order of a push / pop traversal."""
    off = tree.layout()["node_offset"]
    kids = [[] for _ in parent]
    for u, p in enumerate(parent):
        if p >= 0:
            kids[p].append(u)
    calls, stack = [], [(u, False) for u in range(len(parent) - 1, -1, -1) if parent[u] < 0]
    while stack:
        u, pop = stack.pop()
        calls.append((pop, int(off[u]), int(off[u] + seg[u])))
        if not pop:
            stack.append((u, True))
            stack.extend((c, False) for c in reversed(kids[u]))
    return calls


# ---- the contract -----------------------------------------------------------------

def prepare(case, seed):
    parent, seg = _tree(case)
    T, Hq, Hkv, d = int(seg.sum()), case["q_heads"], case["kv_heads"], case["head_dim"]
    kind = torch.float32 if case["dtype"] == F32 else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q, k, v, do = (torch.randn((T, h, d), generator=g, device="cuda", dtype=torch.float32).to(kind)
                   for h in (Hq, Hkv, Hkv, Hq))
    params = dta.AttnParams(Hq, Hkv, d, 1.0 / math.sqrt(d), dta.F32 if case["dtype"] == F32 else dta.BF16)
    state = dict(call=case["call"], params=params, q=q, k=k, v=v, do=do, parent=parent, seg=seg)
    if case["call"] == "step":
        return state            # the pass builds the tree
    tree = state["tree"] = dta.tree_build(parent, seg)
    tree.prepare(params)
    if case["call"] in ("pushpop", "leaforder"):
        if case["call"] == "pushpop":
            state["calls"] = _push_pop_calls(tree, parent, seg)
        else:
            state["calls"] = [(op == dta.OP_BWD, t0, t1)
                              for op, _, t0, t1 in dta.tree_plan(tree, case["block"])["calls"]]
        state["o"], state["dq"] = torch.empty_like(q), torch.empty_like(q)
        state["lse"] = torch.empty((T, Hq), dtype=torch.float32, device="cuda")
        state["dk"] = torch.empty((T, Hkv, d), dtype=torch.float32, device="cuda")
        state["dv"] = torch.empty_like(state["dk"])
        state["ws"] = torch.empty(max(256, dta.workspace_bytes(tree, params, True)), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    s = state
    p, q, k, v, do = s["params"], s["q"], s["k"], s["v"], s["do"]
    if s["call"] in ("pushpop", "leaforder"):
        tree, o, lse, dq, dk, dv = s["tree"], s["o"], s["lse"], s["dq"], s["dk"], s["dv"]
        dk.zero_()
        dv.zero_()
        for backward, t0, t1 in s["calls"]:
            if backward:
                dta.tree_attn_bwd_segment(tree, p, t0, t1, q, k, v, o, lse, do, dq, dk, dv, s["ws"])
            else:
                dta.tree_attn_fwd_segment(tree, p, t0, t1, q, k, v, o, lse)
        return o, lse, dq, dk, dv
    if s["call"] == "step":
        tree = dta.tree_build(s["parent"], s["seg"])
        tree.prepare(p)
    else:
        tree = s["tree"]
    o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
    if s["call"] == "forward":
        return o, lse
    dq, dk, dv = dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do)
    if s["call"] == "step":
        tree.destroy()
    return o, lse, dq, dk, dv


def work(case):
    parent, seg = _tree(case)
    T, Hq, Hkv, d = int(seg.sum()), case["q_heads"], case["kv_heads"], case["head_dim"]
    size = 4 if case["dtype"] == F32 else 2
    pairs = _pairs(parent, seg)
    q_rows, k_rows = T * Hq * d * size, T * Hkv * d * size
    if case["call"] == "forward":   # q, k, v in; o, lse out; two products of head_dim per pair
        return {"bytes": 2 * q_rows + 2 * k_rows + 4 * T * Hq, "flops": pairs * Hq * 4 * d}
    # q, k, v, dO in; o, lse, dq, dk, dv out; two products forward, five backward.  The executors' dk, dv
    # are fp32 whatever the inputs are.
    grads = 2 * T * Hkv * d * (4 if case["call"] in ("pushpop", "leaforder") else size)
    return {"bytes": 4 * q_rows + 2 * k_rows + grads + 4 * T * Hq, "flops": pairs * Hq * 14 * d}


def tolerance(case):
    # About four times the largest error against the same formulas in 64 bits, over the five outputs, measured
    # on the smaller trees above and on a 13 000-token one: bf16 rel 2.5e-3, max 0.15 (P and dS are rounded to
    # bf16 between the products, and the results are); fp32 rel 3.8e-6, max 1.4e-4 (sums of up to 13 000 terms
    # times the heads of a group).
    if case["dtype"] == F32:
        return {"rel": 1e-5, "max": 5e-4}
    return {"rel": 1e-2, "max": 0.5}
