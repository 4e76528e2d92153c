"""The compiled calls on plain tensors against the wrappers' general path, which tensors of
another class still take: the same results, the same refusals."""
import math

import numpy as np
import pytest

import paper_2602_00482_amd as dta
from paper_2602_00482_amd import binding


def _tensors(device, kind, T, Hq, Hkv, d):
    import torch
    g = torch.Generator().manual_seed(3)
    mk = lambda heads: torch.randn((T, heads, d), generator=g).to(kind).to(device)
    return mk(Hq), mk(Hkv), mk(Hkv), mk(Hq)


def test_unknown_arguments_are_left_to_the_general_path():
    import ctypes as C
    import torch
    tree = dta.tree_build([-1, 0], [3, 4])
    p = dta.AttnParams(2, 1, 64, 1.0, dta.F32)
    calls = binding._calls()
    head = (tree.handle.value, C.addressof(p), tree.n_tokens)
    q, k, v, do = _tensors("cpu", torch.float32, 7, 2, 1, 64)
    lse = torch.zeros((7, 2))
    assert calls.fwd(*head, q, k, v, None, None, None) is None              # tensors of the CPU
    assert calls.fwd(*head, q, k, v, None, None) is None                    # too few
    assert calls.fwd(*head, 1, "k", None, None, None, None) is None
    assert calls.bwd(*head, q, k, v, q, lse, do, None, None, None, None) is None
    assert calls.fwd_segment(*head, 0, 3, q, k, v, q, lse) is None
    assert calls.fwd_segment(*head, 1 << 70, 3, q, k, v, q, lse) is None
    assert calls.bwd_segment(*head, 0, 3, q, k, v, q, lse, do, q, k, v, None) is None
    assert calls.fwd(0, 0, 7, q, k, v, None, None, None) is None
    tree.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 2, 128), ("f32", 4, 4, 64)])
def test_compiled_calls_and_general_path_agree(dtype, Hq, Hkv, d):
    import torch

    class Other(torch.Tensor):   # not a plain tensor: the general path
        pass

    parent, seg = np.array([-1, 0, 0], dtype=np.int32), np.array([70, 33, 5], dtype=np.int32)
    T, kind = 108, torch.float32 if dtype == "f32" else torch.bfloat16
    p = dta.AttnParams(Hq, Hkv, d, 1 / math.sqrt(d), dta.F32 if dtype == "f32" else dta.BF16)
    tree = dta.tree_build(parent, seg)
    q, k, v, do = _tensors("cuda", kind, T, Hq, Hkv, d)
    other = q.as_subclass(Other)

    o, lse = dta.tree_attn_fwd(tree, p, other, k, v)
    dq, dk, dv = dta.tree_attn_bwd(tree, p, other, k, v, o, lse, do)
    ref = [t.as_subclass(torch.Tensor) for t in (o, lse, dq, dk, dv)]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
            got = [o, lse, *dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do)]
            assert all(type(t) is torch.Tensor for t in got)
            given = [torch.full_like(t, float("nan")) for t in got]
            ws = torch.empty(max(256, dta.workspace_bytes(tree, p, True)), dtype=torch.uint8, device="cuda")
            res = dta.tree_attn_fwd(tree, p, q, k, v, given[0], given[1])
            res += dta.tree_attn_bwd(tree, p, q, k, v, given[0], given[1], do, *given[2:], ws)
        stream.synchronize()
        for i, (a, b, c, r) in enumerate(zip(ref, got, given, res)):
            assert c is r and torch.equal(a, b) and torch.equal(a, c), i

    seg_out = []
    for first in (other, q):
        o, lse = torch.zeros_like(q), torch.zeros((T, Hq), device="cuda")
        dq, acc = torch.zeros_like(q), [torch.zeros((T, Hkv, d), device="cuda") for _ in range(2)]
        for t0, t1 in ((0, 70), (70, 103), (103, 108)):
            dta.tree_attn_fwd_segment(tree, p, np.int64(t0) if first is other else t0, t1, first, k, v, o, lse)
        for t0, t1 in ((103, 108), (70, 103), (0, 70)):
            dta.tree_attn_bwd_segment(tree, p, t0, t1, first, k, v, o, lse, do, dq, *acc, ws)
        seg_out.append([o, lse, dq, *acc])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*seg_out))

    with pytest.raises(ValueError, match="k: expected"):
        dta.tree_attn_fwd(tree, p, q, k[:, :, :32].contiguous(), v)
    with pytest.raises(ValueError, match="q must be a contiguous"):
        dta.tree_attn_fwd(tree, p, torch.cat((q, q), dim=2)[:, :, :d], k, v)
    with pytest.raises(dta.DtaError, match="dta_tree_attn_fwd_segment"):
        dta.tree_attn_fwd_segment(tree, p, 5, 2000, q, k, v, q, ref[1])
    with pytest.raises(dta.DtaError, match="dta_tree_attn_bwd"):
        dta.tree_attn_bwd(tree, p, q, k, v, ref[0], ref[1], do, workspace=ws[:0])
    tree.destroy()
