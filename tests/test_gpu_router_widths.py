"""The learned router at the widths where its kernel changes (a thread holds 3, 4, 7 or 10 pieces of 512 channels, above 5120
several parts of 8), at widths that do not fill them, and at both ends of the bottleneck, against the oracle."""
import pytest
import torch

import workloads as W
from oracle import router_plus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r,n", [(8, 8, 1), (512, 8, 3), (520, 64, 1), (1544, 16, 2), (2048, 8, 1), (2056, 24, 2), (3584, 64, 1), (5120, 8, 2),
                                   (5128, 8, 1), (12288, 16, 1),
                                   (8192, 64, 1), (8200, 24, 2), (12280, 8, 3)])
def test_router_logits_match_the_oracle(d, r, n):
    import paper_2507_17307_amd as P
    w = W.make_router_weights(d, r, seed=9)
    g = torch.Generator().manual_seed(d + r)
    hidden = torch.randn(n, d, generator=g)
    out = P.binding.new_route_out(n)
    logits = torch.zeros(n, 2, device="cuda")
    P.binding.rs_route_plus(None, hidden.cuda(), n, P.binding.RouterPlus(w.to("cuda")), P.RS_SLM, out, logits)
    torch.cuda.synchronize()
    want = router_plus.router_logits(w, hidden.double())
    # fp32 sums of up to 12288 products in six residual blocks
    assert float((logits.cpu().double() - want).abs().max()) <= 1e-4 * (1 + float(want.abs().max())), (logits, want)
