"""The exponentials behind the records, seen one at a time.  A row with one logit at 0, one at -d and all others far below them has z = 1 in fp32
for d > 17.4 (exp(-d) is less than half an ulp of 1), so its entropy ln z - s / z is the product d exp(-d) and nothing else: the error of the one
exponential and of one rounding."""
import math
from types import SimpleNamespace

import pytest
import torch

from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu

# A product of an exponential rounded to nearest and d is 3.6e-8 from 64 bits in the root mean square (each rounding 2.5e-8, over all
# mantissas), one of an exponential that was rounded twice 4.4e-8.  The estimate from 2048 rows is within 1.6 % of its expectation, one sigma.
RMS = 3.9e-8


def check(h, d):
    """h: entropies of rows with their second logit at -d (fp32), 17.4 < d < 87."""
    d = d.double().cpu()
    want = d * torch.exp(-d)
    rel = (torch.as_tensor(h, dtype=torch.float64) - want) / want
    assert float(rel.square().mean().sqrt()) <= RMS and float(rel.abs().max()) <= 2.5e-7, (float(rel.square().mean().sqrt()), float(rel.abs().max()))


def route(d, vocab):
    import paper_2507_17307_amd as P
    n = d.numel()
    x = torch.full((n, vocab), -150.0, device="cuda")         # exp(-150) is zero in fp32
    x[:, 0], x[:, 1] = 0.0, -d
    out = P.binding.new_route_out(n)
    P.rs_route(x, n, vocab, None, 0.5, P.RS_SLM, out, torch.empty(P.rs_route_scratch_bytes(n, vocab), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert (out[:, 0] == 0).all() and (out[:, 1] & 1 == 0).all()
    return out.view(torch.float32)[:, 2].double().cpu()


# 2048 rows of 33000 entries: one workgroup per row, which is the first to arrive and the last
@pytest.mark.parametrize("n,vocab", [(8192, 4), (4096, 1024), (2048, 33000)])
def test_one_exponential_of_a_row(n, vocab):
    g = torch.Generator(device="cuda").manual_seed(vocab)
    d = torch.empty(n, device="cuda").uniform_(17.5, 86.0, generator=g)
    check(route(d, vocab), d)


@pytest.mark.parametrize("vocab", [4, 33000])
def test_exponentials_below_the_normal_range(vocab):
    """From -87.4 to -103 an fp32 exponential is a multiple of 2^-149 and not yet zero.  It may be one such step off; the product with d is rounded
    once more, by 2^-24 of its value where that is a normal number and half a step where it is not."""
    d = torch.linspace(87.5, 103.0, 300, device="cuda")
    h, dd = route(d, vocab), d.double().cpu()
    want = dd * torch.exp(-dd)
    assert (h > 0).all() and ((h - want).abs() <= (dd + 1) * 2.0 ** -149 + want * 2.0 ** -24).all()


def test_one_exponential_of_a_row_behind_the_lm_head():
    """Many sequences: the softmax states of k_gemm_ring.  Layers of zeros leave the embedding, whose first channel alone the head reads."""
    import paper_2507_17307_amd as P
    n, d, vocab = 128, 128, 8192
    g = torch.Generator().manual_seed(5)
    bf = lambda x: x.to(torch.bfloat16).cuda()  # noqa: E731
    embed = torch.randn(vocab, d, generator=g)
    embed[:, 0] = -10.0                                       # normalised: about -7.5
    head = torch.zeros(vocab, d)
    head[1, 0], head[2:, 0] = 1.0, 16.0
    ones, zeros = torch.ones(d), torch.zeros
    layer = SimpleNamespace(attn_norm=bf(ones), w_qkv=bf(zeros(256, d)), w_o=bf(zeros(d, 128)), mlp_norm=bf(ones), w_gate_up=bf(zeros(256, d)), w_down=bf(zeros(d, 128)))
    w = SimpleNamespace(shape=ModelShape("head", 1, d, 4, 2, 32, 128, vocab, tied_lm_head=False), embed=bf(embed), lm_head=bf(head), final_norm=bf(ones), layers=[layer])
    gpu = P.Model(w, max_ctx=16, max_seqs=n, max_rows=n)
    hs, ds = [], []
    for i in range(16):
        toks = torch.randint(0, vocab, (n,), generator=g).tolist()
        scales = (2.8 + 7.2 * torch.rand(n, generator=g)).tolist()
        got, lg = gpu.decode_step(toks, [0] * n, 0.5, P.RS_SLM, scales, want_logits=True)
        torch.cuda.synchronize()
        assert (lg[:, 0] == 0).all() and float(lg[:, 2:].max()) < -250 and all(r.token == 0 for r in got)
        keep = [k for k in range(n) if 17.5 < -float(lg[k, 1]) < 86]
        hs += [got[k].h_nats for k in keep]
        ds += [-float(lg[k, 1]) for k in keep]
    assert len(hs) > 1500 and math.isfinite(sum(hs))
    check(hs, torch.tensor(ds))


@pytest.mark.parametrize("n,vocab", [(64, 1000), (64, 1001), (64, 32768), (32, 50257), (32, 152064)])
@pytest.mark.parametrize("spread", [0.3, 10.0])
def test_entropy_and_ln_z_of_whole_rows(n, vocab, spread):
    import paper_2507_17307_amd as P
    g = torch.Generator(device="cuda").manual_seed(vocab)
    x = torch.empty(n, vocab, device="cuda").normal_(0, spread, generator=g)
    out = P.binding.new_route_out(n)
    P.rs_route(x, n, vocab, None, 0.5, P.RS_SLM, out, torch.empty(P.rs_route_scratch_bytes(n, vocab), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    h, lz = (out.view(torch.float32)[:, k].double().cpu() for k in (2, 5))
    x = x.double().cpu()
    want = torch.logsumexp(x, 1)
    p = torch.exp(x - want[:, None])
    mean = (p * x).sum(1)
    # ln Z is the largest logit + ln z, the entropy ln z + the mean distance from the largest logit.  z is within a few roundings of 2^-24 of its value (a
    # thread's sums of up to 150 terms, the workgroups'), which is an absolute error of ln z; logarithm, mean and sum add as much of their own values.
    # A distance d is rounded by 2^-24 of it, within a thread and again between threads: so much of its exponential, d times as much of the mean
    top = x.max(1).values
    second = (p * (x - top[:, None]).square()).sum(1)
    assert ((lz - want).abs() <= 2.0 ** -22 * (1 + top.abs() + (want - top))).all()
    assert ((h - (want - mean)).abs() <= 2.0 ** -22 * (1 + (want - top) + (top - mean)) + 2.0 ** -23 * second).all()
