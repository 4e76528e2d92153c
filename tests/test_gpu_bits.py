"""The bf16 kernels' results to the last bit.  Programs compare runs bit by bit, so the order in which a kernel
adds up is no accident: a change that leaves sums in their order must leave these digests alone, and a kernel
that adds in another order on purpose records its own, with what is gained, by `python tests/test_gpu_bits.py`."""
import hashlib
import math
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GOLDEN = os.path.join(ROOT, "tests", "golden", "bf16_bits.txt")
NAMES = ("o", "lse", "dq", "dk", "dv")
CASES = {   # name: parent, seg_len, q heads, kv heads, head_dim
    "small": ([-1, 0, 0], [70, 33, 5], 8, 2, 128),
    "answers d128": ([-1] + [0] * 8, [96, 31, 33, 32, 1, 65, 97, 64, 30], 384, 192, 128),
    "answers d64": ([-1] + [0] * 8, [96, 31, 33, 32, 1, 65, 97, 64, 30], 384, 192, 64),
    "chain": ([-1, 0, 1, 2], [300, 37, 64, 128], 256, 64, 128),
    "two groups": ([-1, 0, 0], [700, 500, 311], 32, 8, 128),
    "long walks": ([-1, 0, 0], [4500, 700, 811], 16, 2, 64),
    # the executors' calls, a push and a pop per node
    "segments small": ([-1, 0, 0], [70, 33, 5], 8, 2, 128),
    "segments": ([-1, 0, 0], [1100, 700, 33], 32, 8, 128),
}


def digests(name):
    import torch
    import paper_2602_00482_amd as dta
    from workloads import make_inputs_numpy
    parent, seg, Hq, Hkv, d = CASES[name]
    x = make_inputs_numpy(int(sum(seg)), Hq, Hkv, d, 61, dtype="bf16")
    q, k, v, do = (torch.from_numpy(x[n]).cuda().to(torch.bfloat16) for n in ("q", "k", "v", "do"))
    p = dta.AttnParams(Hq, Hkv, d, 1.0 / math.sqrt(d), dta.BF16)
    tree = dta.tree_build(np.array(parent, dtype=np.int32), np.array(seg, dtype=np.int32))
    if name.startswith("segments"):
        o, lse, dq = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda"), torch.zeros_like(q)
        acc = [torch.zeros(k.shape, device="cuda") for _ in range(2)]
        ws = torch.empty(dta.workspace_bytes(tree, p, True), dtype=torch.uint8, device="cuda")
        ends = np.cumsum(seg)
        for n, end in zip(seg, ends):
            dta.tree_attn_fwd_segment(tree, p, int(end - n), int(end), q, k, v, o, lse)
        for n, end in zip(seg[::-1], ends[::-1]):
            dta.tree_attn_bwd_segment(tree, p, int(end - n), int(end), q, k, v, o, lse, do, dq, *acc, ws)
        out = (o, lse, dq, *acc)
    else:
        o, lse = dta.tree_attn_fwd(tree, p, q, k, v)
        out = (o, lse, *dta.tree_attn_bwd(tree, p, q, k, v, o, lse, do))
    torch.cuda.synchronize()
    tree.destroy()
    return [hashlib.sha256(t.contiguous().view(torch.uint8).cpu().numpy().tobytes()).hexdigest()[:16] for t in out]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_results_keep_their_bits(name):
    golden = {}
    with open(GOLDEN) as f:
        for line in f:
            case, *rest = line.rstrip("\n").split("\t")
            golden[case] = rest
    got = digests(name)
    assert [n for n, a, b in zip(NAMES, got, golden[name]) if a != b] == []


if __name__ == "__main__":
    sys.path.insert(0, sys.argv[1] if len(sys.argv) > 1 else ROOT)
    for case in CASES:
        print(case, *digests(case), sep="\t", flush=True)
