"""fp32 kernels at the edges of their tiles: launches that fill the chip (one K/V
copy for eight row tiles, dK/dV walks cut into partial sums) on ragged segments,
and launches small enough for the blocks' wave groups to share out the streamed
chunk, where some groups have no rows at all.  Whole tensors against the fp64
oracle at the fp32 bar of the other parity tests (max|err| / max|ref| <= 1e-5)."""
import math

import numpy as np
import pytest

import paper_2602_00482_amd as dta
from oracle import tree_direct as B
from workloads import make_inputs_numpy, random_tree
from parity_util import rel_err, run_hip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,seg", [
    (32, 8, [517, 33, 64, 1, 129, 300, 31]),      # large launch, 4 heads x 2 row blocks of 16
    (32, 2, [600, 15, 257, 96, 65]),              # 16 heads in 2 head blocks, 16-token tiles
    (36, 12, [700, 47, 200, 1]),                  # group of 3: one head per block, 128-token tiles
    (4, 2, [17, 1, 15, 16]),                      # four-wave blocks, walks shorter than one wave group's rows
    (8, 1, [127, 128, 129, 33]),                  # four-wave blocks, edges of the 128-row chunk
    (16, 2, [300, 127, 128, 129, 33]),            # small launch in blocks of eight waves
])
def test_tiles_against_the_oracle(Hq, Hkv, seg, d):
    parent = np.array([-1] + [0] * (len(seg) - 1), dtype=np.int32)
    seg = np.array(seg, dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    tree = dta.tree_build(parent, seg)
    tile = tree.schedule_info(dta.AttnParams(Hq, Hkv, d, scale, dta.F32))["bwd_kv_tile_tokens"]
    tree.destroy()
    # which form the launch takes: blocks that fill the chip, eight-wave and four-wave blocks of a small launch
    assert tile == (128 if Hq > 16 else (32 if d == 64 else 64) // (1 if Hq > 8 else 2)), tile
    x = make_inputs_numpy(T, Hq, Hkv, d, 17, dtype="f32")
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for name, ref in (("o", O), ("lse", LSE), ("dq", dQ), ("dk", dK), ("dv", dV)):
        assert rel_err(got[name], ref) <= 1e-5, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(128, 128), (126, 42), (128, 32), (16, 4), (2, 1)])
def test_rows_do_not_depend_on_keys_they_do_not_see(Hq, Hkv, d):
    """K and V rows that are not finite, of a leaf and of the last token of another one: O and LSE
    of every row that sees none of them are those of finite inputs, in tiles that mix
    the leaves and in the causal tile of a segment call; rows that see them have NaN."""
    import torch
    parent = np.array([-1, 0, 0, 0, 3, 0], dtype=np.int32)
    seg = np.array([70, 33, 21, 50, 64, 77], dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    off = np.concatenate([[0], np.cumsum(seg)])
    x = make_inputs_numpy(T, Hq, Hkv, d, 23, dtype="f32")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    clean = np.ones(T, dtype=bool)
    clean[off[2]:off[3]] = False        # node 2
    clean[T - 1] = False                # last token of node 5
    for r in (*range(off[2], off[3]), T - 1):
        x["v"][r, :, 0], x["v"][r, :, d // 2 + 1], x["v"][r, :, d - 1] = np.nan, np.inf, -np.inf
        x["k"][r, :, 1] = np.inf if r % 2 else np.nan
    t = {n: torch.from_numpy(a).cuda() for n, a in x.items()}
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    o, lse = dta.tree_attn_fwd(tree, p, t["q"], t["k"], t["v"])
    o2, lse2 = torch.zeros_like(o), torch.zeros_like(lse)
    for u in range(len(seg)):
        dta.tree_attn_fwd_segment(tree, p, int(off[u]), int(off[u + 1]), t["q"], t["k"], t["v"], o2, lse2)
    torch.cuda.synchronize()
    tree.destroy()
    for got in ((o, lse), (o2, lse2)):
        for name, a, ref in zip(("o", "lse"), got, (O, LSE)):
            a = a.double().cpu().numpy()
            assert np.isfinite(a[clean]).all(), name
            assert rel_err(a[clean], ref[clean]) <= 1e-5, name
            assert np.isnan(a[~clean]).any(axis=tuple(range(1, a.ndim))).all() or name == "lse", name


@pytest.mark.parametrize("Hq,Hkv,limit_o,limit_dq", [(8, 2, 3.65e-7, 4.82e-7), (64, 16, 3.64e-7, 4.79e-7)])
def test_rounding_errors_of_the_products(Hq, Hkv, limit_o, limit_dq):
    """Relative 2-norm errors against 64 bits, head_dim 128: no larger than those of one
    fused multiply-add chain per quarter of head_dim (four lanes per row on the vector ALU),
    which are the limits here (measured: a small launch, and one that fills the chip).  A product that sums
    head_dim in one chain exceeds them by 5 to 16 %."""
    rng = np.random.default_rng(77)
    seg = np.array([300] + [int(n) for n in rng.integers(60, 300, size=7)], dtype=np.int32)
    parent = np.array([-1] + [0] * 7, dtype=np.int32)
    T, d = int(seg.sum()), 128
    scale = 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 5, dtype="f32")
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    O, _ = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, _, _ = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    err = [float(np.linalg.norm(got[n] - ref) / np.linalg.norm(ref)) for n, ref in (("o", O), ("dq", dQ))]
    print(f"T={T} {Hq}/{Hkv}: o {err[0]:.4e} dq {err[1]:.4e}", flush=True)
    assert err[0] <= limit_o and err[1] <= limit_dq, err


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,sign", [(32, 32, 1), (36, 12, -1), (32, 8, 1), (48, 3, -1)])
def test_forests_in_launches_that_fill_the_chip(Hq, Hkv, sign, d):
    """Tiles that straddle many short nodes, groups of 1, 3, 4 and 16, a negative scale."""
    parent, seg = random_tree(np.random.default_rng(55), 30, 80, n_roots=3)
    T, scale = int(seg.sum()), sign / math.sqrt(d)
    assert T // 16 * Hq >= 2048
    x = make_inputs_numpy(T, Hq, Hkv, d, 62, dtype="f32")
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for name, ref in (("o", O), ("lse", LSE), ("dq", dQ), ("dk", dK), ("dv", dV)):
        assert rel_err(got[name], ref) <= 1e-5, name


# trees for the kernels that multiply fp32 numbers in three bf16 parts: tiles of 128 keys, chunks of 32 rows
PLANES = [
    ([-1], [257], 96, 3),                               # two key tiles and a row, group of 32
    ([-1, 0, 0, 2, 2], [129, 31, 33, 1, 95], 112, 112),     # no groups: row tiles of 128 tokens; edges of the 32-row chunk
    ([-1, -1, 1, 1], [64, 500, 127, 128], 30, 10),          # group of 3
    ([-1, 0, 0, 0], [700, 300, 290, 310], 32, 8),           # cut walks
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("parent,seg,Hq,Hkv", PLANES)
def test_products_in_three_parts(parent, seg, Hq, Hkv, d):
    """Against the oracle, and exact under a change of scale: the parts of 2^n x are 2^n times those of x,
    so outputs linear in V and dO follow them to the last bit."""
    import torch
    parent, seg = np.array(parent, dtype=np.int32), np.array(seg, dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 31, dtype="f32")
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    assert tree.schedule_info(p)["bwd_kv_tile_tokens"] == 128
    t = {n: torch.from_numpy(a).cuda() for n, a in x.items()}

    def run(v, do):
        o, lse = dta.tree_attn_fwd(tree, p, t["q"], t["k"], v)
        return (o, lse, *dta.tree_attn_bwd(tree, p, t["q"], t["k"], v, o, lse, do))

    got = run(t["v"], t["do"])
    refs = (*B.forward(parent, seg, x["q"], x["k"], x["v"], scale),
            *B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale))
    for name, a, ref in zip(("o", "lse", "dq", "dk", "dv"), got, refs):
        assert rel_err(a.double().cpu().numpy(), ref) <= 1e-5, name
    up, down = 2.0 ** 30, 2.0 ** -45
    scaled = run(t["v"] * up, t["do"] * down)
    for name, a, b, f in zip(("o", "lse", "dq", "dk", "dv"), got, scaled, (up, 1, up * down, up * down, down)):
        assert torch.equal(a * f, b), name
    tree.destroy()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(112, 112), (96, 8)])
@pytest.mark.parametrize("what", ["key -inf", "value", "do", "query row"])
def test_numbers_without_three_parts(what, Hq, Hkv, d):
    """Infinities and numbers that bf16 rounds to infinity, in a chunk in the middle of walks or
    in a block's own rows: the results of the fp32 instruction."""
    import torch
    parent = np.array([-1, 0, 0], dtype=np.int32)
    seg = np.array([170, 33, 64], dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 41, dtype="f32")
    big = np.float32(3.395e38)
    if what == "key -inf":            # a score of -inf against every query: the key has no part in any output
        x["q"][:, :, 7] = np.abs(x["q"][:, :, 7]) + 0.1
        x["k"][100, :, 7] = -np.inf
    elif what == "value":
        x["v"][100, :, 3] = big
    elif what == "do":                # (V keeps dP finite)
        x["do"][230, :, 3] = big
        x["v"][:, :, 3] *= 1e-6
        x["k"] *= 1e-3
    else:                             # scores and dK stay finite
        x["q"][[5, 200], :, 9] = big
        x["k"][:, :, 9] *= 1e-38
        x["do"] *= 1e-3
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    assert tree.schedule_info(p)["bwd_kv_tile_tokens"] == 128
    t = {n: torch.from_numpy(a).cuda() for n, a in x.items()}
    o, lse = dta.tree_attn_fwd(tree, p, t["q"], t["k"], t["v"])
    with np.errstate(all="ignore"):
        O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    got, ref = {"o": o, "lse": lse}, {"o": O, "lse": LSE}
    if what in ("do", "query row"):
        got["dq"], got["dk"], got["dv"] = dta.tree_attn_bwd(tree, p, t["q"], t["k"], t["v"], o, lse, t["do"])
        ref["dq"], ref["dk"], ref["dv"] = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for n in got:
        a = got[n].double().cpu().numpy()
        assert np.isfinite(a).all(), n
        assert rel_err(a, ref[n]) <= 1e-5, n
        if what == "value" and n == "o":   # the other columns on their own scale
            cols = [i for i in range(d) if i != 3]
            assert rel_err(a[..., cols], ref[n][..., cols]) <= 1e-5
    tree.destroy()


@pytest.mark.parametrize("Hq,Hkv,d", [(32, 8, 128), (16, 16, 64)])
def test_segment_calls_in_three_parts(Hq, Hkv, d):
    """Forward and backward of a segment behind a prefix that is no multiple of a tile, added to
    accumulators that are not zero."""
    import torch
    parent, seg = np.array([-1, 0], dtype=np.int32), np.array([3301, 1290], dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 51, dtype="f32")
    x["do"][:3301] = 0
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    t = {n: torch.from_numpy(a).cuda() for n, a in x.items()}
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    o, lse = torch.zeros_like(t["q"]), torch.zeros((T, Hq), device="cuda")
    dq = torch.zeros_like(t["q"])
    acc = [torch.full((T, Hkv, d), 1.0, device="cuda") for _ in range(2)]
    ws = torch.empty(dta.workspace_bytes(tree, p, True), dtype=torch.uint8, device="cuda")
    dta.tree_attn_fwd_segment(tree, p, 3301, T, t["q"], t["k"], t["v"], o, lse)
    dta.tree_attn_bwd_segment(tree, p, 3301, T, t["q"], t["k"], t["v"], o, lse, t["do"], dq, *acc, ws)
    tree.destroy()
    for name, a, ref in (("o", o[3301:], O[3301:]), ("lse", lse[3301:], LSE[3301:]), ("dq", dq[3301:], dQ[3301:]),
                         ("dk", acc[0] - 1, dK), ("dv", acc[1] - 1, dV)):
        assert rel_err(a.double().cpu().numpy(), ref) <= 1e-5, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (112, 112), (96, 8)])
def test_a_row_whose_only_key_is_infinite(Hq, Hkv, d):
    """Key 0 has a -inf element against positive queries: every score of row 0 is -inf, though its own
    numbers are finite.  Its LSE is -inf and its output NaN; other rows leave the key out."""
    import torch
    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([170, 33, 64], dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 41, dtype="f32")
    x["q"][:, :, 7] = np.abs(x["q"][:, :, 7]) + 0.1
    x["k"][0, :, 7] = -np.inf
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32", backward=False)
    assert (got["lse"][0] == -np.inf).all() and np.isnan(got["o"][0]).all()
    with np.errstate(all="ignore"):
        O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    assert np.isfinite(got["lse"][1:]).all() and np.isfinite(got["o"][1:]).all()
    assert rel_err(got["lse"][1:], LSE[1:]) <= 1e-5 and rel_err(got["o"][1:], O[1:]) <= 1e-5


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [3e38, -2e30, 1e-37])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (112, 112)])
def test_scales_at_the_ends_of_the_range(Hq, Hkv, scale, d):
    """Scores of ordinary size from a scale near fp32's largest or smallest number."""
    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([170, 33, 64], dtype=np.int32)
    x = make_inputs_numpy(int(seg.sum()), Hq, Hkv, d, 43, dtype="f32")
    f = np.float32(math.sqrt(1 / math.sqrt(d) / abs(scale)))   # q . k scale is that of N(0,1) inputs
    x["q"] *= f
    x["k"] *= f
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    assert rel_err(got["o"], O) <= 1e-5 and rel_err(got["lse"], LSE) <= 1e-5
    dQ, dK, dV = B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)
    for name, ref in (("dq", dQ), ("dk", dK), ("dv", dV)):
        assert rel_err(got[name], ref) <= 1e-5, name


@pytest.mark.parametrize("Hq,Hkv,d,seg,factor,limits", [
    (16, 16, 64, [600, 500, 300, 250], 1, dict(o=2.19e-7, dq=3.71e-7, dk=3.78e-7, dv=3.25e-7)),
    (16, 16, 128, [600, 500, 300, 250], 1, dict(o=2.86e-7, dq=4.38e-7, dk=4.25e-7, dv=3.57e-7)),
    (8, 8, 64, [5000, 700, 900], 1, dict(o=3.16e-7, dq=4.88e-7, dk=4.84e-7, dv=4.29e-7)),   # limits: 4/4 heads
    (4, 4, 128, [5000, 700, 900], 1, dict(o=4.26e-7, dq=5.83e-7, dk=5.49e-7, dv=4.89e-7)),
    # LSE, and the scores of large queries
    (32, 8, 64, [300, 250, 200, 150], 1, dict(o=1.96e-7, lse=4.39e-8)),
    (32, 8, 128, [300, 250, 200, 150], 1, dict(o=2.53e-7, lse=4.37e-8)),
    (32, 8, 64, [300, 250, 200, 150], 30, dict(o=1.03e-6, lse=7.36e-8, dq=4.37e-6, dk=4.39e-6, dv=2.09e-6)),
    (32, 8, 128, [300, 250, 200, 150], 30, dict(o=1.44e-6, lse=9.97e-8, dq=5.99e-6, dk=6.01e-6, dv=3.12e-6)),
    (16, 16, 64, [600, 500, 300, 250], 100, dict(o=2.08e-6, lse=7.40e-8, dq=1.52e-5, dk=1.52e-5, dv=4.83e-6)),
])
def test_errors_of_products_in_three_parts(Hq, Hkv, d, seg, factor, limits):
    """Relative 2-norm errors against 64 bits, of queries `factor` times N(0,1): no larger than those of the
    blocks that share out the keys on the fp32 instruction, which are the limits here (measured)."""
    parent, seg = np.array([-1] + [0] * (len(seg) - 1), dtype=np.int32), np.array(seg, dtype=np.int32)
    T, scale = int(seg.sum()), float(np.float32(1.0 / math.sqrt(d)))
    x = make_inputs_numpy(T, Hq, Hkv, d, 41, dtype="f32")
    x["q"] *= np.float32(factor)
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    ref = dict(zip(("o", "lse"), B.forward(parent, seg, x["q"], x["k"], x["v"], scale)))
    ref.update(zip(("dq", "dk", "dv"), B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)))
    err = {n: float(np.linalg.norm(got[n] - ref[n]) / np.linalg.norm(ref[n])) for n in limits}
    print(f"T={T} {Hq}/{Hkv} d{d}: " + " ".join(f"{n} {e:.3e}" for n, e in err.items()), flush=True)
    assert all(err[n] <= limits[n] for n in limits), err


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("factor", [1e3, 1e5, 3e8])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (112, 112)])
def test_scores_of_any_size(Hq, Hkv, factor, d):
    """Scores of 1e6, 1e10 and 1e17: one key per row has all the weight, but for near ties (in fp32 a score of
    1e17 is known to 1e10), which the seed does without."""
    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([170, 33, 64], dtype=np.int32)
    scale = 1.0 / math.sqrt(d)
    x = make_inputs_numpy(int(seg.sum()), Hq, Hkv, d, 47, dtype="f32")
    x["q"] *= np.float32(factor)
    x["k"] *= np.float32(factor)
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32", backward=False)
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    assert np.isfinite(got["o"]).all() and rel_err(got["lse"], LSE) <= 1e-5
    wrong = np.abs(got["o"] - O).max(axis=-1) > 1e-3
    print(f"rows that differ: {int(wrong.sum())} of {wrong.size}", flush=True)
    assert wrong.mean() <= 1e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (112, 112), (96, 8)])
def test_products_that_overflow(Hq, Hkv, d):
    """Finite numbers whose product is -infinity in fp32: against every key of one query row (LSE -infinity, output
    NaN, no other row touched), and against one key, which then has no weight in any row."""
    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([170, 33, 64], dtype=np.int32)
    T, scale = int(seg.sum()), 1.0 / math.sqrt(d)
    x = make_inputs_numpy(T, Hq, Hkv, d, 53, dtype="f32")
    k = x["k"].copy()
    x["k"][:, :, 7] = -1.234567e30 * (1 + np.abs(k[:, :, 7]))
    x["q"][:, :, 7] = 1.234567e-28
    x["q"][150, :, 7] = 1.234567e30
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32", backward=False)
    assert (got["lse"][150] == -np.inf).all() and np.isnan(got["o"][150]).all()
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    rest = np.arange(T) != 150
    assert rel_err(got["o"][rest], O[rest]) <= 2e-5 and rel_err(got["lse"][rest], LSE[rest]) <= 1e-5
    x["q"][:, :, 7] = 1.234567e20 * (1 + np.abs(k[:, :1, 7]))
    x["k"][:, :, 7] = 0
    x["k"][100, :, 7] = -1.3456e20
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32", backward=False)
    x["k"][100, :, 7] = -1e30   # (so that in 64 bits, too, the key's weight is 0)
    O, LSE = B.forward(parent, seg, x["q"], x["k"], x["v"], scale)
    assert rel_err(got["o"], O) <= 1e-5 and rel_err(got["lse"], LSE) <= 1e-5


LARGE = np.float32(3.0e12)   # beyond 2^40: multiplied on the fp32 instruction


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,parent,seg,rows", [
    (112, 112, [-1, 0, 0], [170, 33, 64], [100]),              # in the middle of a walk
    (96, 8, [-1, 0, 0], [300, 333, 64], [12, 631]),            # in the first chunk, and in a leaf's last key tile
    (32, 8, [-1, 0, 0, 0], [700, 300, 290, 310], [5, 650]),    # dK/dV walks that are cut into partial sums
])
@pytest.mark.parametrize("what", ["k", "v", "q", "do"])
def test_backward_of_numbers_without_three_parts(what, Hq, Hkv, parent, seg, rows, d):
    """One large number in some rows of a tensor, small ones in the same column of the tensor that it is multiplied
    with.  dQ meets the rows of K and V while it streams them and those of Q and dO as its own, dK/dV the other way
    round; in both the walk goes on on the fp32 instruction.  The large column of a gradient and the others
    are compared on scales of their own."""
    parent, seg = np.array(parent, dtype=np.int32), np.array(seg, dtype=np.int32)
    T, scale, col = int(seg.sum()), 1.0 / math.sqrt(d), 9
    x = make_inputs_numpy(T, Hq, Hkv, d, 59, dtype="f32")
    other = {"k": "q", "q": "k", "v": "do", "do": "v"}[what]
    x[what][rows, :, col] = LARGE
    x[other][:, :, col] *= 1 / LARGE
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    info = tree.schedule_info(p)
    tree.destroy()
    assert info["bwd_kv_tile_tokens"] == 128
    if len(seg) == 4:
        assert info["bwd_work_items"] > T // 128 + len(seg)   # some walks are cut
    got = run_hip(parent, seg, x, Hq, Hkv, d, scale, "f32")
    ref = dict(zip(("o", "lse"), B.forward(parent, seg, x["q"], x["k"], x["v"], scale)))
    ref.update(zip(("dq", "dk", "dv"), B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)))
    rest = [i for i in range(d) if i != col]
    for n, r in ref.items():
        assert np.isfinite(got[n]).all(), n
        if n == "lse":
            assert rel_err(got[n], r) <= 1e-5, n
        else:
            assert rel_err(got[n][..., rest], r[..., rest]) <= 1e-5, n
            assert rel_err(got[n][..., col], r[..., col]) <= 1e-5, (n, "large column")


@pytest.mark.parametrize("Hq,Hkv,d,before,rows,limits", [
    (32, 8, 64, 512, 1000, dict(o=6.30e-7, lse=6.25e-8, dq=1.32e-6, dk=1.32e-6, dv=8.87e-7)),
    (32, 8, 128, 512, 1000, dict(o=8.67e-7, lse=8.30e-8, dq=1.78e-6, dk=1.79e-6, dv=1.18e-6)),
    (32, 1, 64, 100, 1100, dict(o=6.29e-7, lse=6.28e-8, dq=1.36e-6, dk=1.75e-6, dv=1.33e-6)),
    (8, 2, 128, 512, 5200, dict(o=1.06e-6, lse=7.95e-8, dq=2.03e-6, dk=2.09e-6, dv=1.47e-6)),
])
def test_errors_of_segment_calls(Hq, Hkv, d, before, rows, limits):
    """Relative 2-norm errors against 64 bits of pushes and pops with queries of 8 times N(0,1), whose scores
    a backward call has to round as the forward did: no larger than in the fp32 kernels that fill the chip or
    share out the keys on the fp32 instruction (measured)."""
    import torch
    parent, seg = np.array([-1, 0], dtype=np.int32), np.array([before, rows], dtype=np.int32)
    T, scale = before + rows, float(np.float32(1.0 / math.sqrt(d)))
    x = make_inputs_numpy(T, Hq, Hkv, d, 41, dtype="f32")
    x["q"] *= np.float32(8)
    t = {n: torch.from_numpy(a).cuda() for n, a in x.items()}
    p = dta.AttnParams(Hq, Hkv, d, scale, dta.F32)
    tree = dta.tree_build(parent, seg)
    o, lse, dq = torch.zeros_like(t["q"]), torch.zeros((T, Hq), device="cuda"), torch.zeros_like(t["q"])
    dk, dv = (torch.zeros((T, Hkv, d), device="cuda") for _ in range(2))
    ws = torch.empty(dta.workspace_bytes(tree, p, True), dtype=torch.uint8, device="cuda")
    for a, b in ((0, before), (before, T)):
        dta.tree_attn_fwd_segment(tree, p, a, b, t["q"], t["k"], t["v"], o, lse)
    for a, b in ((before, T), (0, before)):
        dta.tree_attn_bwd_segment(tree, p, a, b, t["q"], t["k"], t["v"], o, lse, t["do"], dq, dk, dv, ws)
    torch.cuda.synchronize()
    tree.destroy()
    ref = dict(zip(("o", "lse"), B.forward(parent, seg, x["q"], x["k"], x["v"], scale)))
    ref.update(zip(("dq", "dk", "dv"), B.backward(parent, seg, x["q"], x["k"], x["v"], x["do"], scale)))
    err = {n: float(np.linalg.norm(a.double().cpu().numpy() - ref[n]) / np.linalg.norm(ref[n]))
           for n, a in zip(("o", "lse", "dq", "dk", "dv"), (o, lse, dq, dk, dv))}
    print(" ".join(f"{n} {e:.3e}" for n, e in err.items()), flush=True)
    assert all(err[n] <= limits[n] for n in limits), err
