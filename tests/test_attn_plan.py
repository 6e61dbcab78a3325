"""The work split of the walked attention (csrc/attn_plan.h), compiled for the CPU."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_17307_amd", "csrc")
WRAP = """
#include "attn_plan.h"
extern "C" int next_pass(int t0, int t_end) { return rs::walk_next_pass(t0, t_end); }
extern "C" void plan(int n_rows, int n_seqs, int n_kv, int heads, int max_ctx, int n_splits, int n_cu, rs::WalkPlan *out) {
    *out = rs::plan_walk(n_rows, n_seqs, n_kv, heads, max_ctx, n_splits, n_cu);
}
extern "C" int first_len(int total, int longest, int slots, int slices) { return rs::walk_first_len(total, longest, slots, slices); }
extern "C" int try_len(int first, int k) { return rs::walk_try_len(first, k); }
extern "C" int pairs(int n_rows, int n_seqs, int n_kv, int heads, int n_splits, int n_cu) {
    return rs::span_pairs(n_rows, n_seqs, n_kv, heads, n_splits, n_cu);
}
extern "C" int tries() { return rs::WALK_TRIES; }
extern "C" int slots_max() { return rs::WALK_SLOTS_MAX; }
extern "C" int groups_max() { return rs::WALK_GROUPS_MAX; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_plan")
    src, so = d / "wrap.cpp", d / "libattn_plan.so"
    src.write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("t_begin,t_end", [(0, 1), (0, 63), (0, 64), (0, 65), (64, 130), (128, 4562), (4544, 4562), (0, 9157)])
def test_requests_of_a_slice_stay_on_its_pass_grid(lib, t_begin, t_end):
    """Every request starts a whole pass of the slice (16-byte V pieces are aligned there), none lies past the slice, and a
    slice requests each of its passes: once, and the last one once more."""
    starts, t0 = [t_begin], t_begin
    while t0 < t_end:
        starts.append(lib.next_pass(t0, t_end))
        t0 += 64
    passes = list(range(t_begin, t_end, 64))
    assert starts == passes + passes[-1:]


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("walk", "share", "list", "direct", "slices", "groups", "slots", "pieces", "few")]


def split(lib, spans, ctx, n_kv, heads, max_ctx, n_cu=256, max_rows=128):
    """The plan of a call and the pieces (sequence, group, first pass, last pass + 1) that its row table lists: the arithmetic
    of prepare_pieces, one sequence after the other."""
    n, rows, rp = len(spans), sum(spans), 16 // heads
    most = min((max_ctx + 63) // 64, 192, max(512, max_rows * min(72, (max_ctx + 63) // 64)) // rows)
    p = Plan()
    lib.plan(rows, n, n_kv, heads, max_ctx, most, n_cu, ctypes.byref(p))
    if not p.walk:
        return p, None
    groups = [(i, g, -(-(c + min((g + 1) * 4 * rp, s)) // 64)) for i, (s, c) in enumerate(zip(spans, ctx)) for g in range(-(-s // (4 * rp)))]
    if not p.list:
        c = -(-(-(-max(s + c for s, c in zip(spans, ctx)) // p.slices)) // 64)
    else:
        assert len(groups) <= p.groups <= lib.groups_max() and p.slots <= lib.slots_max()
        first = lib.first_len(sum(g[2] for g in groups), max(g[2] for g in groups), p.slots, p.slices)
        tried = [lib.try_len(first, k) for k in range(lib.tries())]
        assert tried[0] == first and tried == sorted(tried) and tried[-1] <= 2 * first
        fits = [t for t in tried if sum(-(-g[2] // t) for g in groups) <= p.slots]
        c = fits[0] if fits else first
    pieces = [(i, g, s, min(s + c, n_p)) for i, g, n_p in groups for s in range(0, n_p, c)]
    return p, pieces


def share(pieces, n_kv, n_cu=256):
    """Passes a workgroup has to walk at least, with two workgroups per CU."""
    return -(-sum(b - a for _, _, a, b in pieces) * n_kv // (2 * n_cu))


BATCHES = [
    # name, KV heads, heads per KV head, max_ctx, spans, contexts
    ("decode, one long context", 4, 7, 4608, [1] * 128, [300] * 127 + [4500]),
    ("decode, one very long context", 4, 7, 10240, [1] * 128, [300] * 64 + [10000] + [300] * 63),
    ("decode of 16, one long context", 4, 7, 9216, [1] * 16, [9000] + [300] * 15),
    ("32 sequences of 2 rows, one long context", 4, 7, 4608, [2] * 32, [300] * 31 + [4500]),
    ("16 x 8 rows", 4, 7, 4608, [8] * 16, [4000] * 16),
    ("8 x 16 rows", 4, 7, 4608, [16] * 8, [4000] * 8),
    ("32 x 2 rows", 4, 7, 4608, [2] * 32, [4000] * 32),
    ("16 x 8 rows, eight KV heads", 8, 5, 9216, [8] * 16, [9000] * 16),
    ("a span of 64 rows beside decode rows", 4, 7, 4608, [64] + [1] * 63, [4000 - 37 * i for i in range(64)]),
    ("32 x 4 rows, two KV heads", 2, 6, 4608, [4] * 32, [4000] * 32),
]


@pytest.mark.parametrize("name,n_kv,heads,max_ctx,spans,ctx", BATCHES, ids=[b[0] for b in BATCHES])
def test_no_workgroup_walks_more_than_twice_the_average_share(lib, name, n_kv, heads, max_ctx, spans, ctx):
    """Unlike contexts, balanced spans, spans beside decode rows: the machine is not left to a few long walks.  (Slices that
    divide the longest context by a number that assumes the longest span for every sequence give 71, 157, 18, 71, 63, 32, 63,
    141, 64 and 63 passes here.)"""
    p, pieces = split(lib, spans, ctx, n_kv, heads, max_ctx)
    assert p.walk and p.list
    longest = -(-max(s + c for s, c in zip(spans, ctx)) // 64)
    assert max(b - a for _, _, a, b in pieces) <= max(2 * share(pieces, n_kv), -(-longest // p.slices))


def test_every_pass_is_in_one_piece_and_the_pieces_fit_their_list(lib):
    rng = random.Random(3)
    listed = 0
    for _ in range(2000):
        n_kv, heads = rng.choice([(1, 8), (2, 6), (4, 7), (8, 5), (8, 1), (4, 2), (32, 1), (2, 4)])
        n = rng.randint(1, 128)
        spans = [1] * n
        for _ in range(rng.choice([0, rng.randint(0, 128 - n)])):
            spans[rng.randrange(n)] += 1
        max_ctx = rng.choice([256, 512, 1024, 2048, 4608, 9216, 12800, 40000])
        ctx = [rng.randint(0, max_ctx - s) if rng.random() < 0.7 else min(300, max_ctx - s) for s in spans]
        p, pieces = split(lib, spans, ctx, n_kv, heads, max_ctx, n_cu=rng.choice([64, 256, 304]))
        if pieces is None:
            continue
        if p.list:
            listed += 1
            assert len(pieces) <= p.pieces
        per_group = {}
        for i, g, a, b in pieces:
            per_group.setdefault((i, g), []).append((a, b))
        for (i, g), parts in per_group.items():
            rp = 16 // heads
            end = -(-(ctx[i] + min((g + 1) * 4 * rp, spans[i])) // 64)
            assert parts[0][0] == 0 and parts[-1][1] == end and all(x[1] == y[0] for x, y in zip(parts, parts[1:]))
            assert len(parts) <= p.slices
        assert len(per_group) == sum(-(-s // (4 * (16 // heads))) for s in spans)
    assert listed > 500


@pytest.mark.parametrize("rows,seqs,n_kv,heads,max_ctx,pairs", [
    (2, 1, 4, 7, 4608, True), (2, 1, 4, 7, 4096, False), (3, 1, 4, 7, 4608, False), (5, 1, 4, 7, 4608, False), (3, 1, 8, 5, 3072, True),
    (4, 1, 8, 5, 3072, False), (3, 2, 2, 6, 4608, True), (4, 2, 2, 6, 4608, True), (2, 1, 2, 6, 4608, False), (2, 1, 2, 6, 9216, True)])
def test_few_rows_past_one_workgroup_per_cu_share_cus(lib, rows, seqs, n_kv, heads, max_ctx, pairs):
    """Calls of two to four rows in one row slot per sequence that are between one and one and a half workgroups per CU."""
    p = Plan()
    lib.plan(rows, seqs, n_kv, heads, max_ctx, max_ctx // 64, 256, ctypes.byref(p))
    assert not p.walk
    assert bool(lib.pairs(rows, seqs, n_kv, heads, max_ctx // 64, 256)) == pairs
