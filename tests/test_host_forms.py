"""Which form of the kernels a call takes (CPU): the rules of dta_tree.cpp at the sizes
where the forms' measured times cross, through the schedule the library reports and
through a small driver around choose_tiles for what it does not report."""
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

import paper_2602_00482_amd as dta

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_00482_amd", "csrc")


@pytest.fixture(scope="module")
def forms():
    """forms(calls), with or without the longest path -> [(q form, dK/dV form, dQ tile, key tile, forward tile where it differs)]"""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    out = os.path.join(tempfile.mkdtemp(prefix="dta_forms_"), "driver")
    cmd = [gxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "host_forms", "driver.cpp"),
           os.path.join(CSRC, "dta_tree.cpp"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def run(calls):
        text = "".join(" ".join(str(int(x)) for x in (*c, 0)[:10]) + "\n" for c in calls)
        res = subprocess.run([out], input=text, capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stderr
        got = [l.split() for l in res.stdout.splitlines()]
        assert len(got) == len(calls)
        return [(q, k, int(bm), int(bn), int(fb)) for q, k, bm, bn, fb in got]

    yield run
    shutil.rmtree(os.path.dirname(out), ignore_errors=True)


def tree_call(parent, seg, Hq, Hkv, d, dtype, backward):
    tree = dta.tree_build(np.asarray(parent, dtype=np.int32), np.asarray(seg, dtype=np.int32))
    info = tree.info()
    tree.destroy()
    T = info["n_tokens"]
    return Hq, Hkv, d, dtype, backward, 0, T, T, info["unique_pairs"], info["max_path_tokens"]


def segment_call(Hq, Hkv, d, backward, before, rows):
    """`rows` rows after `before` tokens of their root path"""
    return Hq, Hkv, d, dta.BF16, backward, 1, rows, before + rows, before * rows + rows * (rows + 1) // 2


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,tokens,small", [
    (16, 1, 2560, True), (16, 1, 12800, False), (16, 1, 24000, False),
    (16, 2, 2560, True), (16, 2, 9600, False), (32, 2, 6400, False), (64, 8, 1600, True), (64, 8, 3100, False),
])
def test_dkdv_tiles_of_a_tree_follow_the_work_of_the_walks(Hq, Hkv, tokens, small, d):
    """One segment: few key tiles, long walks.  The form for launches that leave the chip
    empty (64-key tiles) is 10-30 % slower there once the cut walks fill it."""
    tree = dta.tree_build(np.array([-1], dtype=np.int32), np.array([tokens], dtype=np.int32))
    tile = tree.schedule_info(dta.AttnParams(Hq, Hkv, d, 0.1, dta.BF16))["bwd_kv_tile_tokens"]
    tree.destroy()
    assert (tile == 64) == small, tile


@pytest.mark.parametrize("d", [64, 128])
def test_forms_of_segment_calls(forms, d):
    backward = [   # heads, tokens before, rows, dQ form, dK/dV form
        (16, 1, 9220, 3580, "small", "small"),      # 86 key tiles seen by the average row
        (16, 1, 28420, 3580, "large", "large"),     # 236 of 250
        (16, 1, 54000, 1600, "split", "large"),     # 428, 800 row tiles
        (16, 1, 54000, 600, "small", "small"),      # ... 300 row tiles
        (16, 1, 54000, 3580, "large", "large"),
        (32, 8, 16384, 512, "small", "small"),      # 512 row tiles, a 16K prompt
        (32, 8, 16384, 1024, "split", "large"),     # 1024
        (32, 8, 16384, 1536, "large", "large"),     # 1536
        (64, 8, 2000, 1000, "small", "small"),      # 2000 row tiles, 156 key tiles seen
        (64, 8, 4000, 1000, "small", "small"),      # 281 seen, but blocks of 8 row tiles would be a round and a bit
        (64, 8, 4000, 1600, "large", "large"),      # 300 seen, 3200 row tiles
        (16, 8, 420, 3580, "small", "small"),       # mostly its own causal half
    ]
    got = forms([segment_call(Hq, Hkv, d, 1, before, rows) for Hq, Hkv, before, rows, _, _ in backward])
    for g, c in zip(got, backward):
        assert g[:2] == c[4:], (g, c)
    forward = [   # heads, tokens before, rows, form
        (16, 1, 16384, 1000, "small"), (16, 1, 16384, 2000, "split"), (16, 1, 16384, 2200, "large"),
        (16, 1, 2048, 2200, "split"), (32, 8, 2048, 1500, "large"), (32, 8, 512, 1500, "split"), (4, 4, 8192, 16000, "split"),
        (16, 1, 512, 5000, "large"),
    ]
    got = forms([segment_call(Hq, Hkv, d, 0, before, rows) for Hq, Hkv, before, rows, _ in forward])
    for g, c in zip(got, forward):
        assert g[0] == c[4], (g, c)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("segment", [0, 1])
def test_one_schedule_serves_both_directions(forms, segment, d):
    """The choices of a forward and of a backward call of the same rows describe one schedule, and a
    forward that walks steps finds them there: its tiles are then dQ's."""
    rng = np.random.default_rng(3)
    shapes = []
    for _ in range(400):
        hkv = int(rng.choice([1, 2, 3, 8, 16]))
        hq = hkv * int(rng.choice([1, 2, 3, 4, 5, 8, 16]))
        rows = int(np.exp(rng.uniform(0, np.log(40000))))
        keys = rows + (int(np.exp(rng.uniform(0, np.log(40000)))) if segment else 0)
        pairs = rows * (keys - rows) + rows * (rows + 1) // 2
        shapes.append((hq, hkv, d, int(rng.choice([dta.F32, dta.BF16])), segment, rows, keys, pairs))
    f = forms([s[:4] + (0,) + s[4:] for s in shapes])
    b = forms([s[:4] + (1,) + s[4:] for s in shapes])
    for s, x, y in zip(shapes, f, b):
        assert x[2:] == y[2:], (s, x, y)
        if x[0] in ("small", "tiny"):
            assert y[0] in ("small", "tiny") and x[4] == 0, (s, x, y)


@pytest.mark.parametrize("d", [64, 128])
def test_forms_of_fp32_calls(forms, d):
    """Trees (before = None) and segments on both sides of the measured crossings; both directions take
    one form, and key tiles of 128 say that dK/dV multiplies in three bf16 parts."""
    calls = [   # heads, tokens before, rows, form
        (32, 8, None, 607, "small"), (32, 8, None, 608, "large"), (32, 1, None, 1020, "large"),
        (32, 8, None, 1100, "large"), (32, 8, None, 1290, "large"), (16, 16, None, 9000, "large"),
        (16, 16, 512, 1300, "small"), (32, 8, 4096, 620, "large"), (32, 8, 4096, 500, "small"),
        # segments whose average row sees 53, 64, 82, 97, 93, 97, 190 and 39 key tiles of 128
        (32, 8, 512, 700, "small"), (32, 8, 512, 1000, "small"), (8, 2, 4096, 2400, "small"), (8, 2, 4096, 4200, "large"),
        (32, 8, 1100, 800, "small"), (32, 8, 1160, 800, "large"), (8, 2, 8192, 8000, "large"), (32, 1, 2048, 1700, "small"),
        (32, 1, 2048, 1800, "large"), (8, 2, 512, 5200, "small"), (8, 2, 512, 7100, "large"),   # 3500 row tiles
    ]
    args = []
    for Hq, Hkv, before, rows, _ in calls:
        keys = rows + (before or 0)
        args.append((Hq, Hkv, d, dta.F32, 0, int(before is not None), rows, keys, 1))
    f = forms(args)
    b = forms([a[:4] + (1,) + a[5:] for a in args])
    for c, x, y in zip(calls, f, b):
        assert x == y, (c, x, y)
        assert (x[0].replace("tiny", "small"), x[3] == 128) == (c[4], c[4] == "large"), (c, x)


@pytest.mark.parametrize("Hq,Hkv,d,seg,small", [
    (8, 2, 64, [2401], True), (8, 2, 64, [480, 360, 120, 288, 192, 240, 240, 336, 145], False), (8, 2, 64, [4800], False),
    (16, 16, 64, [1601], True), (32, 8, 64, [651], True), (32, 8, 64, [1001], False), (16, 16, 128, [1200], True), (16, 16, 128, [2000], False),
    (16, 16, 128, [260, 195, 65, 156, 104, 130, 130, 182, 79], False),
])
def test_form_of_an_fp32_tree_follows_its_longest_walk(Hq, Hkv, d, seg, small):
    """1200 row tiles and more: a tree without branches, whose forward is as long as its longest walk, stays in
    blocks that share out the keys until they are a round and a half; a prompt with answers does not."""
    tree = dta.tree_build(np.array([-1] + [0] * (len(seg) - 1), dtype=np.int32), np.array(seg, dtype=np.int32))
    info = tree.schedule_info(dta.AttnParams(Hq, Hkv, d, 0.1, dta.F32))
    tree.destroy()
    assert (info["bwd_kv_tile_tokens"] < 128) == small, info


def test_the_gpu_tests_reach_the_forms_they_name(forms):
    import test_gpu_launch_forms as G
    for tree, Hq, Hkv, _, fwd, dq64, dq128, dkdv in G.FORMS:
        for d, dq in ((64, dq64), (128, dq128)):
            parent, seg = tree()
            f, b = forms([tree_call(parent, seg, Hq, Hkv, d, dta.BF16, way) for way in (0, 1)])
            assert (f[0], b[0], b[1]) == (fwd, dq, dkdv), (Hq, Hkv, d, f, b)
    for dtype, Hq, Hkv, d, dq, dkdv in G.STAGED:
        b = forms([tree_call(*G.staged_tree(), Hq, Hkv, d, dta.F32 if dtype == "f32" else dta.BF16, 1)])[0]
        assert b[:2] == (dq, dkdv), (dtype, Hq, Hkv, d, b)
