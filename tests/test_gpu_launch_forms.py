"""bf16 launches on both sides of the size rules: few rows (or keys) take the form
whose wave groups share out the streamed rows, many take the form that fills the
chip.  Ragged segments at the edges of the 32-, 64- and 128-row tiles, whole
tensors against the fp64 oracle at the bf16 bar (max|err| / max|ref| <= 1e-2)."""
import math

import numpy as np
import pytest

import paper_2602_00482_amd as dta
from oracle import tree_direct as B
from workloads import chain_tree, make_inputs_numpy, random_tree
from parity_util import rel_err, run_hip

pytestmark = pytest.mark.gpu


def _check(seg, Hq, Hkv, d, key_tile, parent=None):
    parent = np.array([-1] + [0] * (len(seg) - 1) if parent is None else parent, dtype=np.int32)
    seg = np.array(seg, dtype=np.int32)
    scale = 1.0 / math.sqrt(d)
    tree = dta.tree_build(parent, seg)
    got_tile = tree.schedule_info(dta.AttnParams(Hq, Hkv, d, scale, dta.BF16))["bwd_kv_tile_tokens"]
    tree.destroy()
    assert got_tile == key_tile, got_tile
    x = make_inputs_numpy(int(seg.sum()), Hq, Hkv, d, 29, dtype="bf16")
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "bf16")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for name, ref in (("o", O), ("lse", LSE), ("dq", dQ), ("dk", dK), ("dv", dV)):
        assert rel_err(got[name], ref) <= 1e-2, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,seg", [
    (4, 2, [17, 1, 31, 33]),                # walks shorter than the groups' rows: some groups stay idle
    (8, 1, [127, 128, 129, 1, 63]),         # eight heads: a step is four heads of one 32-row chunk
    (3, 1, [65, 95, 32, 2]),                # odd group: iterations of two chunks in one step
    (5, 5, [1, 64, 200, 31]),               # no grouping: a step is four chunks
])
def test_small_form(Hq, Hkv, seg, d):
    _check(seg, Hq, Hkv, d, 64)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,seg", [
    (96, 96, [300, 1, 63, 65, 129, 170]),   # no grouping: 256-token query tiles, dQ of head_dim 128 split (128 tokens)
    (128, 64, [257, 33, 310, 95, 31]),       # group of two, dQ of head_dim 128 split
    (256, 64, [300, 127, 128, 129, 40]),    # group of four, blocks of 8 row tiles in both directions
])
def test_large_form(Hq, Hkv, seg, d):
    _check(seg, Hq, Hkv, d, 128)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (4, 2), (3, 3)])
def test_small_form_path_of_many_short_intervals(Hq, Hkv, d):
    """Every second node of the path is preceded by a leaf, so the path is 24 separate
    key intervals of 1 to 70 tokens: steps made of up to four of them, full and ragged."""
    lens = [1, 70, 31, 32, 33, 2, 64, 5, 3, 1, 65, 40, 7, 32, 9, 1, 1, 1, 30, 34, 96, 8, 63, 45]
    parent, seg, tip = [], [], -1
    for n in lens:
        if tip >= 0:
            parent.append(tip)   # a leaf between the tip and the next node of the path
            seg.append(3)
        parent.append(tip)
        seg.append(n)
        tip = len(seg) - 1
    _check(seg, Hq, Hkv, d, 64, parent)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,seg", [
    (30, 10, [257, 33, 310, 95, 31]),       # forward split (660 row tiles): one head per block, 128-token tiles
    (40, 10, [300, 127, 128, 129, 40]),     # ... group of four, 32-token tiles
    (120, 60, [257, 33, 310, 95, 31]),      # backward split at head_dim 128 (2640), group of two
    (128, 16, [300, 1, 63, 65, 129, 170]),  # ... group of eight, two head blocks
    (192, 96, [257, 33, 310, 95, 31]),      # blocks of 8 row tiles in both directions
])
def test_forms_between(Hq, Hkv, seg, d):
    _check(seg, Hq, Hkv, d, 64 if Hq < 100 else 128 if Hkv > 32 else 64)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,rows", [(64, 64, 1000), (64, 64, 993), (48, 16, 700)])
def test_split_segment(Hq, Hkv, rows, d):
    """One segment of 1000 to 2000 row tiles under a ragged prompt, forward and backward,
    against the whole-tree calls (the same pairs: both round P and dS to bf16 once)."""
    import torch
    parent, seg = np.array([-1, 0], dtype=np.int32), np.array([517, rows], dtype=np.int32)
    T, scale = 517 + rows, 1.0 / math.sqrt(d)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, do = (torch.randn((T, Hq, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((T, Hkv, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.BF16)
    tree = dta.tree_build(parent, seg)
    o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
    dq, dk, dv = dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do)
    o2, dq2 = torch.zeros_like(o), torch.zeros_like(dq)
    lse2 = torch.zeros_like(lse)
    dk2, dv2 = torch.zeros(k.shape, device="cuda"), torch.zeros(k.shape, device="cuda")
    ws = torch.empty(max(256, dta.workspace_bytes(tree, p, True)), dtype=torch.uint8, device="cuda")
    for t0, t1 in ((0, 517), (517, T)):
        dta.tree_attn_fwd_segment(tree, p, t0, t1, q, k, v, o2, lse2)
    for t0, t1 in ((517, T), (0, 517)):
        dta.tree_attn_bwd_segment(tree, p, t0, t1, q, k, v, o2, lse2, do, dq2, dk2, dv2, ws)
    for name, a, b in (("o", o2, o), ("lse", lse2, lse), ("dq", dq2, dq), ("dk", dk2, dk), ("dv", dv2, dv)):
        assert rel_err(a.float().cpu().numpy(), b.float().cpu().numpy()) <= 1e-2, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype,Hq,Hkv,n", [
    ("bf16", 4, 2, 300),         # small form
    ("bf16", 40, 10, 500),       # split forward (600 row tiles)
    ("bf16", 128, 32, 500),      # blocks of 8 row tiles
    ("f32", 4, 2, 300), ("f32", 64, 16, 600),
])
def test_a_row_of_infinite_scores(dtype, Hq, Hkv, n, d):
    """One query row whose scores are all -inf (a -inf element against positive keys): its LSE is
    -inf and its output NaN in every form, and no other row changes."""
    import torch
    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([n // 2, n // 4 + 3, n - n // 2 - n // 4 - 3], dtype=np.int32)
    x = make_inputs_numpy(n, Hq, Hkv, d, 41, dtype=dtype)
    x["k"][:, :, 7] = np.abs(x["k"][:, :, 7]) + 0.5
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    p = dta.AttnParams(Hq, Hkv, d, 1.0 / math.sqrt(d), dta.F32 if dtype == "f32" else dta.BF16)
    tree = dta.tree_build(parent, seg)
    t = {k: torch.from_numpy(a).cuda().to(kind) for k, a in x.items()}
    ref = dta.tree_attn_fwd(tree, p, t["q"], t["k"], t["v"])
    row = n - 20
    t["q"][row, :, 7] = -float("inf")
    o, lse = dta.tree_attn_fwd(tree, p, t["q"], t["k"], t["v"])
    torch.cuda.synchronize()
    tree.destroy()
    assert bool((lse[row] == -float("inf")).all()) and bool(torch.isnan(o[row]).all())
    keep = torch.arange(n, device="cuda") != row
    assert torch.equal(o[keep], ref[0][keep]) and torch.equal(lse[keep], ref[1][keep])


def _forest():
    return random_tree(np.random.default_rng(55), 30, 80, n_roots=3)   # 1275 tokens


# (tree, Hq, Hkv, sign of the softmax scale; forms of forward, dQ at head_dim 64 and 128, dK/dV).  That these
# sizes take these forms is checked without a GPU by test_host_forms.py.
FORMS = [
    (_forest, 96, 96, -1, "large", "large", "large", "large"),
    (_forest, 120, 40, 1, "large", "large", "large", "large"),      # groups of 3, 5 and 16
    (_forest, 120, 24, -1, "large", "large", "large", "large"),
    (_forest, 384, 24, 1, "large", "large", "large", "large"),
    (_forest, 72, 24, -1, "large", "large", "split", "large"),
    (_forest, 80, 16, 1, "large", "large", "split", "small"),
    (_forest, 64, 4, -1, "large", "large", "split", "small"),
    (_forest, 44, 44, 1, "large", "split", "split", "large"),
    (_forest, 24, 8, -1, "split", "small", "small", "small"),
    (_forest, 25, 5, 1, "split", "small", "small", "small"),
    (_forest, 16, 1, -1, "split", "small", "small", "small"),
    (_forest, 12, 4, -1, "small", "small", "small", "small"),
    (lambda: (np.array([-1] * 5), np.array([3, 70, 1, 64, 65])), 640, 320, 1, "large", "large", "large", "large"),
    (lambda: chain_tree([300, 37, 64, 128]), 256, 64, 1, "large", "large", "large", "large"),
    # tiles of 256 tokens across two answers: waves leave out chunks of 128 and 64 keys
    (lambda: (np.array([-1, 0, 0]), np.array([500, 640, 511])), 72, 72, 1, "large", "large", "large", "large"),
    # answers that end at and beside 32 rows
    (lambda: (np.array([-1] + [0] * 8), np.array([96, 31, 33, 32, 1, 65, 97, 64, 30])), 384, 192, -1,
     "large", "large", "large", "large"),
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tree,Hq,Hkv,sign", [f[:4] for f in FORMS])
def test_forests_in_every_form(tree, Hq, Hkv, sign, d):
    """Forests whose tiles straddle many short nodes, degenerate trees, odd and large groups
    and a negative scale in the forms that small trees no longer reach."""
    parent, seg = tree()
    T, scale = int(np.sum(seg)), sign / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 61, dtype="bf16")
    got = run_hip(np.asarray(parent, dtype=np.int32), np.asarray(seg, dtype=np.int32), x, Hq, Hkv, d, scale, "bf16")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for name, ref in (("o", O), ("lse", LSE), ("dq", dQ), ("dk", dK), ("dv", dV)):
        assert rel_err(got[name], ref) <= 1e-2, name


# (dtype, Hq, Hkv, d; forms of dQ and dK/dV) on 3848 tokens
STAGED = [("bf16", 64, 16, 128, "large", "large"), ("bf16", 64, 16, 64, "large", "large"),
          ("bf16", 24, 6, 128, "split", "small"), ("bf16", 24, 12, 128, "split", "large"), ("f32", 16, 4, 128, "large", "large"),
          ("f32", 16, 4, 64, "large", "large")]


def staged_tree():
    return random_tree(np.random.default_rng(5), 25, 300, n_roots=2)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [s[:4] for s in STAGED])
def test_stages_one_by_one_give_the_bits_of_one_call(dtype, Hq, Hkv, d):
    """The delta stage as a launch of its own, or inside the dQ launch, in the split form and in
    the forms that fill the chip (the small ones: test_gpu_api.py)."""
    import torch
    parent, seg = staged_tree()
    T = int(seg.sum())
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    q, do = (torch.randn((T, Hq, d), generator=g, device="cuda").to(kind) for _ in range(2))
    k, v = (torch.randn((T, Hkv, d), generator=g, device="cuda").to(kind) for _ in range(2))
    p = dta.AttnParams(Hq, Hkv, d, 1.0 / math.sqrt(d), dta.F32 if dtype == "f32" else dta.BF16)
    tree = dta.tree_build(parent, seg)
    o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
    ref = dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do)
    ws = torch.empty(dta.workspace_bytes(tree, p, True), dtype=torch.uint8, device="cuda")
    for stages in ((dta.BWD_DELTA, dta.BWD_DKDV, dta.BWD_DQ), (dta.BWD_DELTA | dta.BWD_DQ, dta.BWD_DKDV),
                   (dta.BWD_DELTA | dta.BWD_DKDV, dta.BWD_DQ), (dta.BWD_DELTA, dta.BWD_DQ | dta.BWD_DKDV)):
        ws.fill_(0xff)
        out = [torch.full_like(a, float("nan")) for a in ref]
        for st in stages:
            dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do, *out, ws, stages=st)
        torch.cuda.synchronize()
        for a, b in zip(ref, out):
            assert torch.equal(a, b), stages
    tree.destroy()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens", [[40] * 40, [500, 640, 511]])   # chunks of 64 and of 128 keys
def test_skipped_chunks_in_a_forward_that_draws_its_items(lens, d):
    """A forward whose blocks draw their items from queues and whose waves leave out masked chunks: the bits
    of the launch with a block per item, and the oracle's results for two heads."""
    import torch
    H, parent = 512, np.array([-1] * len(lens) if len(lens) > 3 else [-1, 0, 0], dtype=np.int32)
    seg, scale = np.array(lens, dtype=np.int32), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(int(seg.sum()), 2, 2, d, 37, dtype="bf16")
    q, k, v = (torch.from_numpy(x[n]).cuda().to(torch.bfloat16).repeat(1, H // 2, 1) for n in ("q", "k", "v"))
    p = dta.AttnParams(H, H, d, scale, dta.BF16)
    tree = dta.tree_build(parent, seg)
    tiles = tree.schedule_info(p)["fwd_work_items"]
    assert tiles * H >= 8 * 256
    o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
    o2, lse2 = dta.tree_attn_fwd(tree, p, q, k, v, workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    tree.destroy()
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    assert rel_err(o[:, -2:].double().cpu().numpy(), O) <= 1e-2 and rel_err(lse[:, -2:].double().cpu().numpy(), LSE) <= 1e-2
