"""Attention of calls with several rows on caches too long for one 64-position pass per workgroup (k_attn_walk), against
the oracle: slice and pass edges, row slots that straddle the causal edge, every group size in use, one slice without a
merge, rejected sequences, and NaN in every cache row past the contexts."""
import pytest
import torch

import workloads as W
from oracle import decoder, router
from parity import check_invocation
from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu

# name, query heads, KV heads, head_dim, max_ctx, contexts, rows of every sequence (None: one each)
CASES = [
    ("decode_g7_hd128", 14, 2, 128, 4608, [0, 63, 64, 4607, 577], None),
    ("decode_g1_hd64", 4, 4, 64, 3000, [2999, 128, 1, 127, 2000], None),
    ("decode_g8_hd32", 8, 1, 32, 12800, [12799, 6400, 9000], None),                  # longer than 192 slices of one pass
    ("decode_one_slice", 8, 4, 32, 256, [(37 * i) % 256 for i in range(100)], None),  # no merge kernel
    ("short_spans_share_a_slot", 12, 4, 128, 4608, [100, 4600, 63], [2, 3, 1]),
    ("spans_g7_hd128", 14, 2, 128, 4608, [4480], [128]),
    ("spans_g3_hd128", 6, 2, 128, 2048, [1, 1990, 700, 0], [17, 58, 1, 40]),
    ("spans_g8_hd64", 8, 1, 64, 9216, [9000, 64, 3000], [60, 2, 66]),
    ("spans_g1_hd32", 4, 4, 32, 4096, [4000, 4095, 63, 62], [64, 1, 16, 33]),
]


@pytest.mark.parametrize("name,nq,nkv,hd,max_ctx,ctx,rows", CASES, ids=[c[0] for c in CASES])
def test_walked_attention_matches_the_oracle(name, nq, nkv, hd, max_ctx, ctx, rows):
    import paper_2507_17307_amd as P
    shape = ModelShape(name, 1, 256, nq, nkv, hd, 256, 512, tied_lm_head=False)
    w = W.make_weights(shape, 31, 1)
    n = len(ctx)
    rows = rows or [1] * n
    gpu = P.Model(w.to("cuda"), max_ctx=max_ctx, max_seqs=n + 1, max_rows=128)
    ref = decoder.OracleModel(w, max_ctx, n_slots=n)
    slots = [(i * 3 + 1) % n if n % 3 else i for i in range(n)]
    g = torch.Generator().manual_seed(7)
    gpu.kv_view("k").fill_(float("nan"))
    gpu.kv_view("v").fill_(float("nan"))
    for i in range(n):
        for which, cache in (("k", ref.k_cache), ("v", ref.v_cache)):
            x = torch.randn(1, nkv, ctx[i], hd, generator=g).bfloat16()
            gpu.kv_view(which)[:, slots[i], :, :ctx[i]] = x.cuda()
            cache[:, slots[i], :, :ctx[i]] = x.double()
    toks = [W.rng.randint(31, 50 + i, 0, rows[i], shape.vocab).tolist() for i in range(n)]
    scales = [1.0 + i % 4 for i in range(n)]
    if rows == [1] * n:
        got, lg = gpu.decode_step([t[0] for t in toks], ctx, 0.6, P.RS_SLM, scales, slots, want_logits=True)
    else:
        got, lg = gpu.catchup_prefill(toks, ctx, 0.6, P.RS_SLM, scales, slots, want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        want = ref.forward(toks[i], ctx[i], slot=slots[i], logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{name} sequence {i}")
    if rows == [1] * n:
        # a rejected sequence beside valid ones
        got, lg = gpu.decode_step([t[0] for t in toks] + [1], list(ctx) + [max_ctx], 0.6, P.RS_SLM, scales + [1.0], slots + [n],
                                  want_logits=True)
        torch.cuda.synchronize()
        assert got[n].flags & P.FLAG_BADARG and not any(r.flags & P.FLAG_BADARG for r in got[:n])
        for i in range(n):
            want = ref.forward(toks[i], ctx[i], slot=slots[i], logit_scale=scales[i])["logits"]
            check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{name} sequence {i} beside a rejected one")
