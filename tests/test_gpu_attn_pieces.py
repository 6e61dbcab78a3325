"""Walked attention of several sequences, whose pieces the row table lists (attn_plan.h): unlike contexts, balanced spans, spans
beside decode rows, rows with one slice beside rows with many, rejected sequences; against the oracle."""
import pytest
import torch

import test_gpu_attn_walk as walk

pytestmark = pytest.mark.gpu

# name, query heads, KV heads, head_dim, max_ctx, contexts, rows of every sequence (None: one each)
CASES = [
    ("one_long_context_g2_hd32", 8, 4, 32, 4608, [70 - i for i in range(39)] + [4500], None),
    ("decode_17_passes", 8, 4, 32, 1088, [(53 * i) % 1088 for i in range(100)], None),                      # just past the fixed split
    ("decode_16_passes_one_slice", 8, 4, 32, 1024, [(53 * i) % 1024 for i in range(100)], None),
    ("more_than_128_slices", 8, 1, 32, 12800, [12000, 9000, 63], None),
    ("pairs_of_rows_g7_hd128", 14, 2, 128, 2048, [2046, 63, 64, 62, 0, 127, 128, 1000] + [20 * i for i in range(16)], [2] * 24),
    ("balanced_spans_g7_hd128", 14, 2, 128, 2048, [1900, 1800, 1700, 1600, 1500, 1400], [8] * 6),
    ("span_beside_decode_rows", 12, 4, 64, 2048, [1024] + [100 * i for i in range(15)], [64] + [1] * 15),
    ("rows_on_both_sides_of_a_slice_edge", 6, 2, 128, 4608, [60, 120, 190, 250, 4000, 57], [10] * 6),
]


@pytest.mark.parametrize("name,nq,nkv,hd,max_ctx,ctx,rows", CASES, ids=[c[0] for c in CASES])
def test_listed_pieces_match_the_oracle(name, nq, nkv, hd, max_ctx, ctx, rows):
    walk.test_walked_attention_matches_the_oracle(name, nq, nkv, hd, max_ctx, ctx, rows)


@pytest.mark.parametrize("name,nq,nkv,hd,max_ctx,ctx,rows", [
    ("slice_edges_g7_hd128", 14, 2, 128, 4608, [60, 120, 190, 250, 4000, 57], [10] * 6),
    ("slice_edges_two_passes_g6_hd128", 12, 2, 128, 1024, [127, 125, 120, 255, 63] + [(71 * i) % 1000 for i in range(35)], [5, 4, 3, 5, 2] + [2] * 35),
    ("slice_edges_g8_hd64", 8, 1, 64, 9216, [9000, 60, 3000], [60, 10, 56]),
    ("one_sequence_g7_hd128", 14, 2, 128, 4608, [50], [128]),
], ids=lambda v: v if isinstance(v, str) else "")
def test_every_row_of_a_span_is_right_at_slice_edges(name, nq, nkv, hd, max_ctx, ctx, rows):
    """Spans whose first rows have one slice and whose last ones more: the outputs of all rows, through the K/V rows that the
    second layer makes of them (logits come from the last row only)."""
    import paper_2507_17307_amd as P
    import workloads as W
    from oracle import decoder, router
    from parity import check_invocation
    from workloads.shapes import ModelShape
    shape = ModelShape(name, 2, 256, nq, nkv, hd, 256, 512, tied_lm_head=False)
    w = W.make_weights(shape, 31, 1)
    n = len(ctx)
    gpu = P.Model(w.to("cuda"), max_ctx=max_ctx, max_seqs=n, max_rows=128)
    ref = decoder.OracleModel(w, max_ctx, n_slots=n)
    g = torch.Generator().manual_seed(7)
    for i in range(n):
        for which, cache in (("k", ref.k_cache), ("v", ref.v_cache)):
            x = torch.randn(2, nkv, ctx[i], hd, generator=g).bfloat16()
            gpu.kv_view(which)[:, i, :, :ctx[i]] = x.cuda()
            cache[:, i, :, :ctx[i]] = x.double()
    toks = [W.rng.randint(31, 50 + i, 0, rows[i], shape.vocab).tolist() for i in range(n)]
    got, lg = gpu.catchup_prefill(toks, ctx, 0.6, P.RS_SLM, [2.0] * n, list(range(n)), want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        want = ref.forward(toks[i], ctx[i], slot=i, logit_scale=2.0)["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{name} sequence {i}")
        for which, cache in (("k", ref.k_cache), ("v", ref.v_cache)):
            a = gpu.kv_view(which)[1, i, :, ctx[i]:ctx[i] + rows[i]].cpu().double()
            b = cache[1, i, :, ctx[i]:ctx[i] + rows[i]].double()
            # bf16 values of nearly equal fp32 sums: one rounding step (2^-8 of the value) apart at most, and a little for values near 0
            assert float(((a - b).abs() - b.abs() * 2.0 ** -7).max()) <= 1e-3, (name, which, i)


@pytest.mark.parametrize("bad_seq", [0, 3, 5])
@pytest.mark.parametrize("fault", ["slot", "position", "token", "same slot"])
def test_a_rejected_sequence_of_a_catch_up_leaves_the_others_alone(bad_seq, fault):
    """Six spans on a long cache, one of them (the first, one inside, the last) out of range: its record is flagged, its
    cache rows are not written, and the others are what they are without it."""
    import paper_2507_17307_amd as P
    import workloads as W
    from oracle import decoder, router
    from parity import check_invocation
    from workloads.shapes import ModelShape
    shape = ModelShape("rejected", 1, 256, 14, 2, 128, 256, 512, tied_lm_head=False)
    w = W.make_weights(shape, 37, 1)
    spans, ctx, max_ctx = [3, 9, 1, 8, 2, 20], [4000, 63, 128, 2500, 4606, 70], 4608
    n = len(spans)
    gpu = P.Model(w.to("cuda"), max_ctx=max_ctx, max_seqs=n + 1, max_rows=64)
    ref = decoder.OracleModel(w, max_ctx, n_slots=n)
    g = torch.Generator().manual_seed(11)
    for i in range(n):
        for which, cache in (("k", ref.k_cache), ("v", ref.v_cache)):
            x = torch.randn(1, shape.n_kv_heads, ctx[i], shape.head_dim, generator=g).bfloat16()
            gpu.kv_view(which)[:, i, :, :ctx[i]] = x.cuda()
            cache[:, i, :, :ctx[i]] = x.double()
    toks = [W.rng.randint(37, 60 + i, 0, spans[i], shape.vocab).tolist() for i in range(n)]
    slots, pos, given = list(range(n)), list(ctx), [list(t) for t in toks]
    rejected = {bad_seq}
    if fault == "slot":
        slots[bad_seq] = n + 1
    elif fault == "position":
        pos[bad_seq] = max_ctx - spans[bad_seq] + 1
    elif fault == "token":
        given[bad_seq][-1] = shape.vocab
    else:
        slots[bad_seq] = slots[(bad_seq + 1) % n]                 # both that name the slot are rejected
        rejected.add((bad_seq + 1) % n)
    before = gpu.kv_view("k").clone()
    got, lg = gpu.catchup_prefill(given, pos, 0.6, P.RS_SLM, [2.0] * n, slots, want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        if i in rejected:
            assert got[i].flags & P.FLAG_BADARG and got[i].token == -1, (i, got[i])
            assert torch.equal(gpu.kv_view("k")[:, i], before[:, i]), i
        else:
            want = ref.forward(toks[i], ctx[i], slot=i, logit_scale=2.0)["logits"]
            check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"sequence {i} beside a rejected one")


@pytest.mark.parametrize("table", [[1, 5, 9, 12], [0, 5, 5, 12], [0, 9, 5, 12], [0, 5, 9, 11], [0, 5, 9, 13], [0, -4, 9, 12]])
def test_a_malformed_offset_table_rejects_every_sequence(table):
    import paper_2507_17307_amd as P
    import workloads as W
    from workloads.shapes import ModelShape
    shape = ModelShape("malformed", 1, 256, 14, 2, 128, 256, 512, tied_lm_head=False)
    gpu = P.Model(W.make_weights(shape, 37, 1).to("cuda"), max_ctx=4608, max_seqs=3, max_rows=16)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    before = gpu.kv_view("k").clone()
    out = P.binding.new_route_out(3)
    P.rs_catchup_prefill(gpu.handle, 3, 12, i32([0, 1, 2]), i32(list(range(12))), i32(table), i32([4000, 70, 0]), None, 0.6, P.RS_SLM, out, None)
    torch.cuda.synchronize()
    for r in P.binding.read_route_out(out):
        assert r.flags & P.FLAG_BADARG and r.token == -1
    assert torch.equal(gpu.kv_view("k"), before)


@pytest.mark.parametrize("name,nq,nkv,hd,max_ctx,ctx,rows", [
    ("two_pairs_g7_hd128", 14, 2, 128, 4608, [4400, 70], [2, 2]),
    ("one_and_two_rows_g7_hd128", 14, 2, 128, 4608, [100, 4606], [1, 2]),
    ("three_rows_g5_hd64", 10, 2, 64, 8448, [8383], [3]),
    ("four_rows_g4_hd32", 16, 4, 32, 5120, [62], [4]),
], ids=lambda v: v if isinstance(v, str) else "")
def test_few_rows_past_one_workgroup_per_cu_match_the_oracle(name, nq, nkv, hd, max_ctx, ctx, rows):
    """k_attn_span built for two workgroups per CU: two to four rows, more workgroups than CUs but too few to walk."""
    walk.test_walked_attention_matches_the_oracle(name, nq, nkv, hd, max_ctx, ctx, rows)


def test_replayed_calls_list_the_pieces_of_their_own_contexts():
    """A call whose buffers repeat is replayed from a graph: the pieces have to follow the positions that the buffers hold at that
    time.  Contexts of two kinds in turn, with eager work in between, against plain launches (the legacy stream)."""
    import paper_2507_17307_amd as P
    import workloads as W
    from workloads.shapes import ModelShape
    shape = ModelShape("replays", 2, 256, 14, 2, 128, 256, 512, tied_lm_head=False)
    n, max_ctx = 24, 4608
    gpu = P.Model(W.make_weights(shape, 39, 1).to("cuda"), max_ctx=max_ctx, max_seqs=n, max_rows=n)
    g = torch.Generator(device="cuda").manual_seed(3)
    gpu.kv_k.normal_(generator=g)
    gpu.kv_v.normal_(generator=g)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    contexts = [i32([4500] + [70] * (n - 1)), i32([64 * i + 1000 for i in range(n)])]
    slot, tok, pos = i32(list(range(n))), i32([7 * i % 512 for i in range(n)]), i32([0] * n)
    out, logits = P.binding.new_route_out(n), torch.zeros(n, shape.vocab, device="cuda")
    side = torch.cuda.Stream()

    def call(ctx, stream):
        pos.copy_(ctx)
        logits.zero_()
        torch.cuda.synchronize()
        P.rs_decode_step(gpu.handle, n, slot, tok, pos, None, 0.6, P.RS_SLM, out, logits, stream)
        torch.cuda.synchronize()
        return logits.clone()

    # a call of one kind writes K/V rows inside the other kind's contexts: after two passes over them the caches no longer change
    for _ in range(2):
        for c in contexts:
            call(c, 0)
    want = [call(c, 0) for c in contexts]
    assert not torch.equal(want[0], want[1])
    for k in range(8):                                        # plain, captured, replays
        assert torch.equal(call(contexts[k % 2], side), want[k % 2]), k
