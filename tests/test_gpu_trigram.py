"""Full 2-gram contexts with dense weights on the clustered kernels (trigram_kernels.hpp): every
instantiation and the edges of its range against the float64 oracle.  Tolerances are those of
test_gpu_parity: distances 1e-5 relative, marginals 1e-5 absolute, paths bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev, library_option
from test_gpu_tables_local import both_orders
from test_gpu_parity import check_path, check_posteriors, forbid_arcs

pytestmark = pytest.mark.gpu


# V: 3 is the smallest label set taken; 11, 12 the last with one workgroup an item and the first with two;
# 19/20, 35/36, 42/43, 64 the edges of the instantiations; 32 and 28 whole and ragged shares of the labels;
# B = 20 at V = 32 takes the wide workgroups, B = 140 more items than clusters
@pytest.mark.parametrize("V,T,B", [(3, 9, 2), (11, 9, 3), (12, 8, 3), (19, 7, 2), (20, 7, 2), (28, 9, 5), (32, 20, 3),
                                   (32, 6, 20), (35, 5, 2), (36, 5, 2), (42, 5, 2), (43, 4, 2), (64, 4, 3),
                                   (20, 5, 140)])
def test_every_instantiation(V, T, B):
    announce("clustered trigram", V, T, B)
    cfg = workloads.dense(B=B, T=T, V=V, order=2, sigma=1.5, seed=100 + V, len_lo=max(1, T - 3), len_hi=T)
    check_posteriors(cfg, order=2)
    check_path(cfg, order=2)
    dist = lb.last_shortest_distance(dev(cfg["w"]), dev(cfg["lengths"]), order=2)
    assert_dist_close(dist.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 2)[1])


@pytest.mark.parametrize("V", [2, 7, 65])
def test_one_workgroup_kernels_keep_the_rest(V):
    announce("trigram, one workgroup per item, V", V)
    cfg = workloads.dense(B=2, T=5, V=V, order=2, sigma=1.0, seed=V, len_lo=3, len_hi=5)
    with library_option(lb.OPT_FORCE_SOLO, 1):
        check_posteriors(cfg, order=2)
        check_path(cfg, order=2)
    if V != 7:
        check_posteriors(cfg, order=2)
        check_path(cfg, order=2)


@pytest.mark.parametrize("V", [5, 32, 44])
def test_lengths_status_scale_and_accumulate(V):
    announce("trigram: lengths 0, 1, 2, T, invalid; scale and accumulate, V", V)
    T = 7
    cfg = workloads.dense(B=6, T=T, V=V, order=2, sigma=1.0, seed=9 + V)
    cfg["lengths"] = np.array([0, 1, 2, T, T + 1, -1], np.int32)
    cfg["w"][1, 1:] = np.nan                                   # frames past the length are not read into a result
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    status = torch.full((6,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(w, lengths, order=2, item_status=status)
    assert status.cpu().tolist() == [0, 0, 0, 0, 1, 1]
    ok = dict(w=cfg["w"][:4], lengths=cfg["lengths"][:4])
    _, D_o = oracle.forward(ok["w"], ok["lengths"], 2)
    g_o = oracle.posteriors(ok["w"], ok["lengths"], 2)
    assert_dist_close(D.cpu().numpy()[:4], D_o)
    assert np.all(np.isnan(D.cpu().numpy()[4:])) and torch.all(g[4:] == 0)
    assert np.max(np.abs(g.cpu().numpy()[:4] - g_o)) <= TOL_POST_ABS
    dist = lb.last_shortest_distance(w, lengths, order=2).cpu().numpy()
    assert_dist_close(dist[:4], D_o)
    assert np.all(np.isnan(dist[4:]))
    labels, states, score = lb.last_shortest_path(w, lengths, order=2)
    l_o, s_o, sc_o = oracle.viterbi(ok["w"], ok["lengths"], 2, "f32")
    assert np.array_equal(labels.cpu().numpy()[:4], l_o) and np.array_equal(states.cpu().numpy()[:4], s_o)
    assert torch.all(labels[4:] == -1) and torch.all(states[4:] == -1)
    base = torch.full_like(w, 0.5)
    lb.last_arc_posteriors(w, lengths, order=2, dw=base, scale=-2.0, accumulate=True)
    want = 0.5 - 2.0 * g
    for b in range(6):
        n = int(cfg["lengths"][b])
        want[b, n if 0 <= n <= T else 0:] = 0.5
    assert torch.max(torch.abs(base - want)).item() < 1e-6


@pytest.mark.parametrize("V", [9, 21, 46])
def test_ties_and_forbidden_arcs(V):
    announce("trigram: integer weights with ties, forbidden arcs, V", V)
    rng = np.random.default_rng(V)
    C = workloads.num_states(V, 2)
    wc = rng.integers(-1, 2, size=(2, 7, C, V + 1)).astype(np.float32)
    check_path(dict(w=wc, lengths=np.array([7, 4], np.int32), B=2), order=2)
    check_path(dict(w=np.zeros((1, 4, C, V + 1), np.float32), lengths=np.array([4], np.int32), B=1), order=2)
    # (sigma 4: scores of up to 30 in base 2, three float32 roundings of at most 1e-6 each in a marginal's exponent)
    cfg = workloads.dense(B=2, T=6, V=V, order=2, sigma=4.0, seed=V)
    check_path(forbid_arcs(cfg, 5), order=2)
    check_posteriors(cfg, order=2)
    cfg["w"][rng.random(cfg["w"].shape) < 0.3] = -np.inf       # arcs that do not exist
    check_path(cfg, order=2)
    check_posteriors(cfg, order=2)


def test_bounded_waits_end_and_flag():
    announce("trigram: a spin limit of one poll")
    cfg = workloads.dense(B=3, T=30, V=24, order=2, sigma=1.0, seed=4)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    _, D_o = oracle.forward(cfg["w"], cfg["lengths"], 2)
    status = torch.full((3,), -1, dtype=torch.int32, device="cuda")
    with library_option(lb.OPT_SPIN_LIMIT, 1):
        D, _ = lb.last_arc_posteriors(w, lengths, order=2, item_status=status)
        torch.cuda.synchronize()
        D, st = D.cpu().numpy(), status.cpu().numpy()
        for b in range(3):
            assert st[b] in (0, 5)
            if st[b] == 5:
                assert np.isnan(D[b])
            else:
                assert abs(D[b] - D_o[b]) <= 1e-5 * abs(D_o[b])
        lb.last_shortest_path(w, lengths, order=2, item_status=status)
        torch.cuda.synchronize()
        assert all(s in (0, 5) for s in status.cpu().tolist())
    check_posteriors(cfg, order=2)
    check_path(cfg, order=2)


# V: one, two, fourteen and sixteen workgroups an item and direction
@pytest.mark.parametrize("V", [5, 24, 42, 64])
def test_items_whose_waits_ran_out_are_computed_all_the_same(V):
    announce("trigram: a spin limit of one poll, results and status as ever, V", V)
    T = 8 if V > 40 else 20
    cfg = workloads.dense(B=4, T=T, V=V, order=2, sigma=1.0, seed=40 + V, len_lo=T - 3, len_hi=T)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    _, D_o = oracle.forward(cfg["w"], cfg["lengths"], 2)
    g_o = oracle.posteriors(cfg["w"], cfg["lengths"], 2)
    status = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    with library_option(lb.OPT_SPIN_LIMIT, 1):
        check_posteriors(cfg, order=2)
        check_path(cfg, order=2)
        base = torch.full_like(w, 0.5)
        D, _ = lb.last_arc_posteriors(w, lengths, order=2, dw=base, scale=-2.0, accumulate=True, item_status=status)
        assert status.cpu().tolist() == [0] * 4
        assert_dist_close(D.cpu().numpy(), D_o)
        assert np.max(np.abs(base.cpu().numpy() - (0.5 - 2.0 * g_o))) <= 2.0 * TOL_POST_ABS
        assert_dist_close(lb.last_shortest_distance(w, lengths, order=2, item_status=status).cpu().numpy(), D_o)
        assert status.cpu().tolist() == [0] * 4
        best = lb.last_shortest_distance(w, lengths, order=2, semiring="tropical", item_status=status)
        assert status.cpu().tolist() == [0] * 4
        assert np.array_equal(best.cpu().numpy(), oracle.viterbi(cfg["w"], cfg["lengths"], 2, "f32")[2])


@pytest.mark.parametrize("V,B", [(24, 8), (50, 20)])
def test_calls_on_several_streams_share_the_chip(V, B):
    announce("trigram: three calls at a time on streams of their own, V, B", V, B)
    cfg = workloads.dense(B=B, T=12, V=V, order=2, sigma=1.0, seed=V, len_lo=9, len_hi=12)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    D, g = lb.last_arc_posteriors(w, lengths, order=2)
    labels, states, score = lb.last_shortest_path(w, lengths, order=2)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for _ in range(2):
        status = [torch.full((B,), -1, dtype=torch.int32, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        out = []
        for i, stream in enumerate(streams):
            with torch.cuda.stream(stream):
                out.append(lb.last_shortest_path(w, lengths, order=2, item_status=status[i]) if i == 1
                           else lb.last_arc_posteriors(w, lengths, order=2, item_status=status[i]))
        torch.cuda.synchronize()
        assert all(torch.all(x == 0) for x in status)
        for i in (0, 2):                     # (an item that another kernel had to take agrees within the tolerance)
            assert_dist_close(out[i][0].cpu().numpy(), D.cpu().numpy())
            assert torch.max(torch.abs(out[i][1] - g)).item() <= TOL_POST_ABS
        assert torch.equal(out[1][0], labels) and torch.equal(out[1][1], states) and torch.equal(out[1][2], score)


# 4161 states: slices of 755 items; 4096 states of a table: of 768
@pytest.mark.parametrize("order,V,C,B", [(2, 64, 4161, 800), (0, 3, 4096, 1600)])
def test_distance_of_a_batch_in_slices(order, V, C, B):
    announce("distance of a batch whose vectors take more than 24 MiB: order, V, B", order, V, B)
    T = 2 if order else 3
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    w = torch.randn((B, T, C, V + 1), generator=g, device="cuda")
    lengths = torch.randint(0, T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lengths[-2] = T + 1
    o_order, g_order = (order, order) if order else both_orders(workloads.random_table(C, V, seed=C))
    some = [0, 1, B // 2, 700, 754, 755, 756, 767, 768, 769, B - 1]
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    D = lb.last_shortest_distance(w, lengths, order=g_order, item_status=status)
    best = lb.last_shortest_distance(w, lengths, order=g_order, semiring="tropical")
    assert status.cpu().tolist() == [0] * (B - 2) + [1, 0]
    assert torch.isnan(D[-2]) and torch.isfinite(D[:-2]).all()
    w_o, l_o = w[some].cpu().numpy(), lengths[some].cpu().numpy()
    assert_dist_close(D[some].cpu().numpy(), oracle.forward(w_o, l_o, o_order)[1])
    assert np.array_equal(best[some].cpu().numpy(), oracle.viterbi(w_o, l_o, o_order, "f32")[2])
    with library_option(lb.OPT_FORCE_SOLO, 1):                 # the general kernels on the whole batch
        again = lb.last_shortest_distance(w, lengths, order=g_order)
    assert_dist_close(D.cpu().numpy()[:-2], again.cpu().numpy()[:-2])


# clusters of 22 to 32 workgroups, the two directions of an item on two XCDs (up to four items); with more items both
# directions on one XCD again
@pytest.mark.parametrize("V,T,B", [(43, 6, 4), (43, 4, 9), (51, 5, 3), (63, 4, 1), (64, 5, 4), (47, 4, 5), (64, 3, 9)])
def test_directions_on_two_xcds(V, T, B):
    announce("clustered trigram, directions apart", V, T, B)
    cfg = workloads.dense(B=B, T=T, V=V, order=2, sigma=1.5, seed=300 + V, len_lo=1, len_hi=T)
    check_posteriors(cfg, order=2)
    check_path(cfg, order=2)
    dist = lb.last_shortest_distance(dev(cfg["w"]), dev(cfg["lengths"]), order=2)
    assert_dist_close(dist.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 2)[1])


def test_calls_on_several_streams_with_directions_on_two_xcds():
    test_calls_on_several_streams_share_the_chip(60, 4)
