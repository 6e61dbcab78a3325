"""k_gemm_ring where it can go wrong: blocks of 4, 8 and 16 rows on matrices that take it from three rows on, an LM head of up to
three sequences in blocks of four rows, waves with one and with two row blocks, four and eight of them, vocabularies whose last tile is ragged, a
matrix of two windows of K (fewer than the rings hold), a head of fewer groups than CUs, the widest groups, and the order of its sums."""
import dataclasses

import pytest
import torch

import workloads as W
from oracle import decoder, router
from parity import check_invocation
from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu

BIG = ModelShape("ring_big", 1, 3072, 24, 8, 128, 11264, 20503, tied_lm_head=True)      # gate/up, down and LM head: 64 MB and more
WIDE = ModelShape("ring_wide", 1, 1536, 12, 2, 128, 27648, 1000, tied_lm_head=False)
NARROW = ModelShape("ring_narrow", 1, 1536, 12, 2, 128, 8960, 1000, tied_lm_head=False)


@pytest.fixture(scope="module")
def big():
    return W.make_weights(BIG, 53, 1)


def run(w, shape, spans, slots, max_ctx, where):
    """One call of spans[i] rows per sequence, the first token at position 0, checked against the oracle."""
    import paper_2507_17307_amd as P
    n, rows = len(spans), sum(spans)
    gpu = P.Model(w.to("cuda"), max_ctx=max_ctx, max_seqs=max(slots) + 1, max_rows=rows)
    ref = decoder.OracleModel(w, max_ctx, n_slots=max(slots) + 1)
    toks = W.rng.randint(53, rows, 0, rows, shape.vocab).tolist()
    cut = [toks[sum(spans[:i]):sum(spans[:i + 1])] for i in range(n)]
    scales = [1.0 + i % 5 for i in range(n)]
    got, lg = gpu.catchup_prefill(cut, [0] * n, 0.6, P.RS_SLM, scales, slots, want_logits=True)
    torch.cuda.synchronize()
    for i in sorted({0, n // 2, n - 1}):
        want = ref.forward(cut[i], 0, slot=slots[i], logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{where}, sequence {i}")


@pytest.mark.parametrize("spans", [[3], [2, 2], [2, 1, 2], [8], [9], [1, 2, 3, 4, 6], [70], [30, 51]])
def test_rows_of_a_large_matrix(spans, big):
    run(big, BIG, spans, list(range(len(spans))), 96, f"spans {spans}")


@pytest.fixture(scope="module")
def narrow():
    return W.make_weights(NARROW, 57, 1)


@pytest.mark.parametrize("spans", [[65], [40, 41], [128]])
def test_narrow_groups_of_many_rows(spans, narrow):
    """Eight multiplying waves of one row block, some without rows: groups of three tiles (down) and of five (gate/up)."""
    run(narrow, NARROW, spans, list(range(len(spans))), 136, f"spans {spans}")


@pytest.fixture(scope="module")
def wide():
    return W.make_weights(WIDE, 71, 1)


@pytest.mark.parametrize("rows", [81, 97, 128])
def test_widest_groups_of_many_rows(rows, wide):
    """Gate/up in groups of 14 tiles above 64 rows (as on the 32B width): X one window ahead, W two; waves with one row block and with two."""
    run(wide, WIDE, [rows], [0], 136, f"{rows} rows")


def call(weights, n, max_ctx=16):
    """A decode step of n sequences at position 0 (attention to one position is the value row itself): logits, K and V of every layer."""
    import paper_2507_17307_amd as P
    m = P.Model(weights, max_ctx=max_ctx, max_seqs=16, max_rows=16)
    toks = W.rng.randint(73, 1, 0, 16, 1000).tolist()[:n]
    _, lg = m.decode_step(toks, [0] * n, 0.6, P.RS_SLM, [1.0 + i % 5 for i in range(n)], want_logits=True)
    torch.cuda.synchronize()
    return lg.clone(), m.kv_view("k")[:, :n, :, 0].clone(), m.kv_view("v")[:, :n, :, 0].clone()


@pytest.mark.parametrize("n", [3, 5, 8, 16])
def test_the_order_of_sums_of_an_lm_head_is_the_same_on_both_kernels(n):
    """1279 column tiles stay on k_gemm_rows, 1280 take the ring: the logits that both have are the same bits."""
    shape = ModelShape("order_head", 1, 2176, 8, 2, 64, 384, 20480, tied_lm_head=False)
    w = W.make_weights(shape, 73, 1, device="cuda")
    below = dataclasses.replace(w, shape=dataclasses.replace(shape, vocab=20464), embed=w.embed[:20464].contiguous(), lm_head=w.lm_head[:20464].contiguous())
    (a, ka, va), (b, kb, vb) = call(w, n), call(below, n)
    assert torch.equal(a[:, :20464], b) and torch.equal(ka, kb) and torch.equal(va, vb)


def test_the_order_of_sums_of_a_layer_is_the_same_on_both_kernels():
    """A down projection that k_gemm_rows takes at 4 rows and the ring at 5 (ring_layer): the second layer's K and V and the logits are the same bits."""
    shape = ModelShape("order_layer", 2, 3584, 28, 4, 128, 16896, 1000, tied_lm_head=False)
    w = W.make_weights(shape, 79, 1, device="cuda")
    (a, ka, va), (b, kb, vb) = call(w, 4), call(w, 5)
    assert torch.equal(a, b[:4]) and torch.equal(ka, kb[:, :4]) and torch.equal(va, vb[:, :4])


@pytest.mark.parametrize("vocab", [65, 8196, 8197])
@pytest.mark.parametrize("n", [17, 66, 97])
def test_lm_head_of_few_tiles(vocab, n):
    shape = ModelShape("ring_head", 1, 128, 4, 2, 32, 128, vocab, tied_lm_head=False)
    run(W.make_weights(shape, 59, 1), shape, [1] * (n - 1) + [2], list(range(n)), 16, f"{n} sequences")


@pytest.mark.parametrize("d, heads, hd", [(128, 4, 32), (1152, 4, 32), (2176, 8, 128)])
def test_rotary_of_ragged_workgroups(d, heads, hd):
    """Rotary items around the 256 of a workgroup, a rejected sequence among the rows."""
    import paper_2507_17307_amd as P
    shape = ModelShape("chunks", 2, d, heads, 2, hd, 256, 1000, tied_lm_head=False)
    w = W.make_weights(shape, 61, 1)
    n = 5
    gpu = P.Model(w.to("cuda"), max_ctx=16, max_seqs=n, max_rows=n)
    ref = decoder.OracleModel(w, 16, n_slots=n)
    toks = W.rng.randint(61, n, 0, n, shape.vocab).tolist()
    toks[2] = shape.vocab                                                  # out of range: this sequence alone is flagged
    scales = [1.0 + i % 5 for i in range(n)]
    got, lg = gpu.decode_step(toks, [0] * n, 0.6, P.RS_SLM, scales, want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        if i == 2:
            assert got[i].flags & P.FLAG_BADARG, got[i]
            continue
        want = ref.forward([toks[i]], 0, slot=i, logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"width {d}, sequence {i}")


@pytest.mark.parametrize("vocab", [1004, 1005])
def test_logits_of_a_buffer_at_any_address(vocab):
    """Quads of logits leave in one store where vocabulary and address allow it: the same values wherever the buffer starts, nothing outside."""
    import paper_2507_17307_amd as P
    n = 18
    shape = ModelShape("ring_logits", 1, 128, 4, 2, 32, 128, vocab, tied_lm_head=False)
    gpu = P.Model(W.make_weights(shape, 67, 1).to("cuda"), max_ctx=16, max_seqs=n, max_rows=n)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    slot, pos, tok = i32(list(range(n))), i32([0] * n), i32(W.rng.randint(67, n, 0, n, vocab).tolist())
    scale, out = torch.ones(n, device="cuda"), P.binding.new_route_out(n)
    got = []
    for first in (4, 5, 7):
        buf = torch.full((n * vocab + 16,), 7.0, device="cuda")
        lg = buf[first:first + n * vocab].view(n, vocab)
        P.rs_decode_step(gpu.handle, n, slot, tok, pos, scale, 0.6, P.RS_SLM, out, lg)
        torch.cuda.synchronize()
        assert (buf[:first] == 7.0).all() and (buf[first + n * vocab:] == 7.0).all()
        got.append(lg.clone())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
