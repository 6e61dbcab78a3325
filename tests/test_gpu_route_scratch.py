"""rs_route on long rows counts the arrivals of its workgroups in the caller's scratch, which nobody has cleared: the records do not depend on
what it held before, on calls that shared it, or on a graph that replays the call."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(n, vocab):
    g = torch.Generator(device="cuda").manual_seed(n * 7 + vocab)
    return torch.randn(n, vocab, generator=g, device="cuda") * 2, torch.rand(n, generator=g, device="cuda") * 6 + 0.5


@pytest.mark.parametrize("n,vocab", [(1, 32769), (3, 50257), (2, 152064), (17, 131073), (64, 33000), (128, 40004)])
def test_any_scratch_gives_the_same_records(n, vocab):
    import paper_2507_17307_amd as P
    x, scale = _inputs(n, vocab)
    out = P.binding.new_route_out(n)
    size = P.rs_route_scratch_bytes(n, vocab)
    want = None
    for fill in (0, 0xFF, 0x01, None):
        scratch = torch.full((size,), fill, dtype=torch.uint8, device="cuda") if fill is not None else torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda")
        for _ in range(3):                                    # the second call finds what the first one left
            out.fill_(-1)
            P.rs_route(x, n, vocab, scale, 0.5, P.RS_SLM, out, scratch)
            got = out.clone()
            want = got if want is None else want
            assert torch.equal(got, want), fill
    # another shape on the same scratch in between
    m = max(1, n // 2)
    small = P.binding.new_route_out(m)
    P.rs_route(x, m, vocab, scale, 0.5, P.RS_SLM, small, scratch)
    out.fill_(-1)
    P.rs_route(x, n, vocab, scale, 0.5, P.RS_SLM, out, scratch)
    assert torch.equal(out, want)


def test_a_replayed_call_routes_what_its_buffer_holds():
    import paper_2507_17307_amd as P
    n, vocab = 5, 152064
    x, scale = _inputs(n, vocab)
    other = torch.randn_like(x)
    out, eager = P.binding.new_route_out(n), P.binding.new_route_out(n)
    scratch, scratch2 = (torch.full((P.rs_route_scratch_bytes(n, vocab),), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2))
    P.rs_route(x, n, vocab, scale, 0.5, P.RS_SLM, out, scratch)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.rs_route(x, n, vocab, scale, 0.5, P.RS_SLM, out, scratch)
    for i in range(4):
        x.add_(other, alpha=0.25)
        out.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        P.rs_route(x, n, vocab, scale, 0.5, P.RS_SLM, eager, scratch2)
        assert torch.equal(out, eager), i
