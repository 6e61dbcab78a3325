"""Row norms of multi-row calls at the widths where a thread holds another number of quads (4096, 8192 and 12288 values a row), with partial sums
of the projection before them and, for the final norm, with gathered rows."""
import pytest
import torch

import workloads as W
from oracle import decoder, router
from parity import check_invocation
from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu


# 4096: one quad a thread; 4224 and 8192: two, the second partly filled and full; 8320 and 12288: three
@pytest.mark.parametrize("d", [4096, 4224, 8192, 8320, 12288])
@pytest.mark.parametrize("spans", [[5], [1, 9, 10]])
def test_a_layer_of_any_width_matches_the_oracle(d, spans):
    import paper_2507_17307_amd as P
    # O and down split over workgroups (16 and 32 windows of K), so both norms after them add partial sums
    shape = ModelShape("wide", 1, d, 16, 2, 64, 2048, 512, tied_lm_head=False)
    w = W.make_weights(shape, 89, 1)
    n = len(spans)
    gpu = P.Model(w.to("cuda"), max_ctx=16, max_seqs=n, max_rows=sum(spans))
    ref = decoder.OracleModel(w, 16, n_slots=n)
    toks = [W.rng.randint(89, i, 0, s, shape.vocab).tolist() for i, s in enumerate(spans)]
    scales = [1.0 + i for i in range(n)]
    got, lg = gpu.catchup_prefill(toks, [0] * n, 0.6, P.RS_SLM, scales, want_logits=True)
    torch.cuda.synchronize()
    for i in range(n):
        want = ref.forward(toks[i], 0, slot=i, logit_scale=scales[i])["logits"]
        check_invocation(got[i], lg[i], want, 0.6, router.SLM, where=f"width {d}, sequence {i}")
        # a K or V rounded the other way (2^-8 of one of 64 channels) moves a logit of a context of ten by up to 1e-3 of its size; a quad that a norm
        # leaves out moves it by that quad's share of the row, at least sqrt(4 / 12288) = 2e-2
        assert float((lg[i].cpu().double() - want).norm()) <= 4e-3 * float(want.norm())
