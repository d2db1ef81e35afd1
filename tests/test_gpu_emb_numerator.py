"""The numerator of a loss on on-the-fly weights behind the weights kernel (shapes of 10^8 hidden units and more) and beside it (smaller
ones): the results of the two calls by themselves, and captured into a graph."""
import pytest
import torch

from paper_2304_13134_amd import binding as lb
from gpu_util import announce

pytestmark = pytest.mark.gpu


def inputs(B, T, V, H, U):
    g = torch.Generator(device="cuda")
    g.manual_seed(B + T + V)
    C = 1 + V + V * V
    f = torch.randn((B, T, H), generator=g, device="cuda").bfloat16()
    e = (0.5 * torch.randn((C, H), generator=g, device="cuda")).bfloat16()
    W = (torch.randn((H, V + 1), generator=g, device="cuda") / H ** 0.5).bfloat16()
    lengths = torch.randint(T // 2, T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    refs = torch.randint(1, V + 1, (B, U), generator=g, device="cuda", dtype=torch.int32)
    ulen = torch.randint(0, U + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    return lb.SharedEmb(f, e, W), lengths, refs, ulen


# hidden units 0.97e8, 1.02e8, 3e8
@pytest.mark.parametrize("B,T,V,H,U", [(2, 90, 32, 512, 20), (2, 95, 32, 512, 20), (4, 280, 32, 256, 70)])
def test_loss_is_distance_and_numerator_and_replays(B, T, V, H, U):
    announce("on-the-fly loss, numerator beside and behind the weights:", B, T, V, H, U)
    se, lengths, refs, ulen = inputs(B, T, V, H, U)
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    D0 = lb.last_shortest_distance(se, lengths, order=2)
    N0 = lb.last_intersect_reference(se, lengths, refs, ulen, order=2)
    D, N, grads = lb.last_globally_normalized_loss(se, lengths, refs, ulen, order=2, item_status=status)
    assert torch.equal(D, D0) and torch.equal(N, N0) and torch.all(status == 0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    out = tuple(torch.empty_like(x) for x in grads)
    with torch.cuda.graph(graph):
        d, n, _ = lb.last_globally_normalized_loss(se, lengths, refs, ulen, order=2, dw=out, item_status=status)
    for _ in range(3):
        for x in (d, n, *out):
            x.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(d, D0) and torch.equal(n, N0)
        for x, y in zip(out, grads):                   # (cells are added up with atomics: float32 sums in another order)
            assert float((x - y).abs().max()) <= 1e-5 * float(y.abs().max())
        float(torch.randn(1000, device="cuda").sum())     # eager work between the replays
