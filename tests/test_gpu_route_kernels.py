"""rs_route at the sizes where its kernels change: one workgroup per row up to 32768 entries, partial states above, rows that are not a
multiple of four entries, several rows per launch, masked entries (the most negative value the router takes as finite), ties."""
import math

import pytest
import torch

from oracle import router

pytestmark = pytest.mark.gpu

CASES = [(1, 2), (3, 5), (1, 63), (2, 4096), (5, 4097), (1, 32768), (3, 32765), (2, 32769), (2, 32772), (64, 33001), (128, 40000), (9, 152064)]


def route(x, scale, tau=0.5):
    import paper_2507_17307_amd as P
    n, v = x.shape
    out = P.binding.new_route_out(n)
    P.rs_route(x, n, v, scale, tau, P.RS_SLM, out, torch.empty(P.rs_route_scratch_bytes(n, v), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return P.binding.read_route_out(out)


@pytest.mark.parametrize("n,vocab", CASES)
@pytest.mark.parametrize("masked", [False, True])
def test_records_match_the_oracle(n, vocab, masked):
    g = torch.Generator().manual_seed(n * 100003 + vocab)
    x = torch.randn(n, vocab, generator=g) * 1.5
    if masked:                                                # whole stretches of a row, so that some threads see nothing else
        keep = torch.randint(0, vocab, (n,), generator=g)
        far = (torch.arange(vocab)[None] - keep[:, None]).abs() > max(1, vocab // 50)
        x[far] = -3.0e38
    scale = None if masked else torch.rand(n, generator=g) * 6 + 0.5
    got = route(x.cuda(), None if scale is None else scale.cuda())
    for i in range(n):
        row = x[i].double() * (1.0 if scale is None else float(scale[i]))
        want = router.route(row, 0.5, router.SLM)
        # fp32 products with the scale and sums of up to 1.5e5 exponentials: a few ulp of the largest logit and of ln V
        assert abs(got[i].h_nats - want["h_nats"]) <= 2e-4 and abs(got[i].log_z - want["log_z"]) <= 1e-4, (i, got[i], want)
        assert abs(got[i].h_norm - want["h_nats"] / math.log(vocab)) <= 2e-4
        assert got[i].token == want["token"], (i, got[i], want)


@pytest.mark.parametrize("vocab", [1000, 1001, 40000])
def test_ties_take_the_lowest_index_and_bad_values_are_flagged(vocab):
    import paper_2507_17307_amd as P
    x = torch.zeros(4, vocab)
    x[0, [vocab - 1, vocab // 2, 7]] = 3.0
    x[1, vocab - 1] = float("nan")
    x[2, 3] = float("-inf")
    got = route(x.cuda(), None)
    assert got[0].token == 7 and got[3].token == 0 and abs(got[3].h_nats - math.log(vocab)) <= 1e-4
    for i in (1, 2):
        assert got[i].flags & P.FLAG_NONFINITE and got[i].token == -1 and math.isnan(got[i].h_nats)
