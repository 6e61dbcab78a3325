"""Calls of 3 .. 128 rows on the matrix-core kernels: the activation buffers between them hold blocks of 1, 2, 4, 8 or 16 rows in
operand order (frag_index), so every row count around those block sizes, as a span and as decode rows, against the oracle.
The first shape's projections have too few columns for k_gemm_ring (ring_layer) and stay on k_gemm_rows, whatever the row count;
those of the second take it from 17 rows on (gate/up from 3), with two waves per row block up to 32 rows, one up to 64, and above 64
two row blocks per wave or, in narrow groups, eight waves of one."""
import pytest
import torch

import workloads as W
from oracle import decoder, router
from parity import check_invocation
from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu

SHAPE = ModelShape("operand_order", 1, 2176, 8, 2, 64, 384, 1000, tied_lm_head=False)     # wider than 2048: three rows take them too


@pytest.fixture(scope="module")
def weights():
    return W.make_weights(SHAPE, 41, 1)


@pytest.mark.parametrize("rows", [3, 4, 5, 8, 9, 15, 16, 17, 33])
def test_row_counts_around_the_block_sizes(rows, weights):
    import paper_2507_17307_amd as P
    gpu = P.Model(weights.to("cuda"), max_ctx=64, max_seqs=rows, max_rows=rows)
    ref = decoder.OracleModel(weights, 64, n_slots=rows)
    toks = W.rng.randint(41, rows, 0, 2 * rows, SHAPE.vocab).tolist()
    got, lg = gpu.catchup_prefill([toks[:rows]], [0], 0.6, P.RS_SLM, [2.0], [rows - 1], want_logits=True)
    torch.cuda.synchronize()
    check_invocation(got[0], lg[0], ref.forward(toks[:rows], 0, slot=rows - 1, logit_scale=2.0)["logits"], 0.6, router.SLM, where=f"span of {rows}")
    scales = [1.0 + i % 5 for i in range(rows)]
    pos = [0] * (rows - 1) + [rows]
    got, lg = gpu.decode_step(toks[rows:], pos, 0.6, P.RS_SLM, scales, want_logits=True)
    torch.cuda.synchronize()
    for i in range(rows):
        want = ref.forward([toks[rows + i]], pos[i], slot=i, logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{rows} sequences, {i}")


@pytest.mark.parametrize("n", [18, 40, 65, 128])
def test_lm_head_of_many_sequences_with_thirteen_column_tiles(n):
    """A vocabulary of 3328 column tiles (the last one ragged) on 256 CUs: workgroups of 13 tiles, split between two waves up to 32
    sequences, on four waves up to 64 and on eight above (which row counts take 13 is checked in test_gemm_plan.py)."""
    import paper_2507_17307_amd as P
    shape = ModelShape("wide_vocab", 1, 128, 4, 2, 32, 128, 53233, tied_lm_head=False)
    w = W.make_weights(shape, 43, 1)
    gpu = P.Model(w.to("cuda"), max_ctx=16, max_seqs=n, max_rows=n)
    ref = decoder.OracleModel(w, 16, n_slots=n)
    toks = W.rng.randint(43, n, 0, n, shape.vocab).tolist()
    scales = [1.0 + i % 5 for i in range(n)]
    got, lg = gpu.decode_step(toks, [0] * n, 0.6, P.RS_SLM, scales, want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        want = ref.forward([toks[i]], 0, slot=i, logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"sequence {i} of {n}")


TILE_SHAPE = ModelShape("tile_kernel", 1, 3072, 24, 8, 128, 10240, 1000, tied_lm_head=False)


@pytest.fixture(scope="module")
def tile_weights():
    return W.make_weights(TILE_SHAPE, 47, 1)


@pytest.mark.parametrize("rows", [16, 17, 32, 33, 64, 65, 128])
def test_row_counts_around_the_wave_arrangements_of_the_tile_kernel(rows, tile_weights):
    import paper_2507_17307_amd as P
    w = tile_weights
    gpu = P.Model(w.to("cuda"), max_ctx=136, max_seqs=rows, max_rows=rows)
    ref = decoder.OracleModel(w, 136, n_slots=rows)
    toks = W.rng.randint(47, rows, 0, 2 * rows, TILE_SHAPE.vocab).tolist()
    got, lg = gpu.catchup_prefill([toks[:rows]], [0], 0.6, P.RS_SLM, [2.0], [rows - 1], want_logits=True)
    torch.cuda.synchronize()
    check_invocation(got[0], lg[0], ref.forward(toks[:rows], 0, slot=rows - 1, logit_scale=2.0)["logits"], 0.6, router.SLM, where=f"span of {rows}")
    pos = [0] * (rows - 1) + [rows]
    scales = [1.0 + i % 5 for i in range(rows)]
    got, lg = gpu.decode_step(toks[rows:], pos, 0.6, P.RS_SLM, scales, want_logits=True)
    torch.cuda.synchronize()
    for i in sorted({0, 15, min(16, rows - 1), rows // 2, rows - 1}):          # rows at the edges of 16-row blocks
        want = ref.forward([toks[rows + i]], pos[i], slot=i, logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"{rows} sequences, {i}")
