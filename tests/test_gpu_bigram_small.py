"""Full 1-gram contexts of 4 to 96 states (bigram_kernels.hpp) against the float64 oracle, at the edges
of its tiles; tolerances of test_gpu_parity."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev, library_option
from test_gpu_parity import check_path, check_posteriors

pytestmark = pytest.mark.gpu


# V = C - 1: up to 3 labels stay in the log domain, 96 lies just outside; 31/32, 47/48, 63/64, 95 the edges of the
# instantiations; 34 and 61 rows that no 16-byte piece divides
@pytest.mark.parametrize("V", [1, 2, 3, 4, 7, 31, 32, 34, 47, 48, 61, 63, 64, 95, 96])
def test_sizes_and_lengths(V):
    announce("small bigram, V", V)
    cfg = workloads.dense(B=8, T=9, V=V, order=1, sigma=1.5, seed=200 + V)
    cfg["lengths"] = np.array([0, 1, 2, 3, 4, 7, 8, 9], np.int32)
    cfg["w"][1, 1:] = np.nan                                   # frames past the length are not read into a result
    check_posteriors(cfg)
    check_path(cfg)
    dist = lb.last_shortest_distance(dev(cfg["w"]), dev(cfg["lengths"]))
    assert_dist_close(dist.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 1)[1])


@pytest.mark.parametrize("V", [3, 32, 70])
def test_long_batch_and_older_kernels(V):
    announce("small bigram, 40 items of 60 frames, V", V)
    cfg = workloads.dense(B=40, T=60, V=V, order=1, sigma=1.0, seed=V, len_lo=40, len_hi=60)
    check_posteriors(cfg)
    check_path(cfg)
    for generation in (1, 2):                                  # the clustered kernels stay selectable here
        with library_option(lb.OPT_CLUSTER_GENERATION, generation):
            check_posteriors(cfg)
    for mode in (0, 2):
        with library_option(lb.OPT_CLUSTER_VITERBI, mode):
            check_path(cfg)


@pytest.mark.parametrize("V", [5, 33, 80])
def test_status_scale_and_accumulate(V):
    announce("small bigram: invalid lengths, scale, accumulate, V", V)
    T = 7
    cfg = workloads.dense(B=4, T=T, V=V, order=1, seed=9 + V)
    cfg["lengths"] = np.array([T, T + 1, -1, 3], np.int32)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    status = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(w, lengths, item_status=status)
    assert status.cpu().tolist() == [0, 1, 1, 0]
    assert torch.isnan(D[1:3]).all() and torch.all(g[1:3] == 0)
    assert torch.isnan(lb.last_shortest_distance(w, lengths, item_status=status)[1:3]).all()
    assert status.cpu().tolist() == [0, 1, 1, 0]
    labels, states, score = lb.last_shortest_path(w, lengths, item_status=status)
    assert status.cpu().tolist() == [0, 1, 1, 0]
    assert torch.all(labels[1:3] == -1) and torch.all(states[1:3] == -1) and torch.isnan(score[1:3]).all()
    base = torch.full_like(w, 0.5)
    lb.last_arc_posteriors(w, lengths, dw=base, scale=-2.0, accumulate=True)
    want = 0.5 - 2.0 * g
    want[3, 3:] = 0.5
    want[1:3] = 0.5
    assert torch.max(torch.abs(base - want)).item() < 1e-6


@pytest.mark.parametrize("V", [4, 40, 90])
def test_ties_missing_arcs_and_range(V):
    announce("small bigram: ties, arcs of weight -inf and -1e4, wide range, V", V)
    rng = np.random.default_rng(V)
    C = V + 1
    check_path(dict(w=rng.integers(-1, 2, size=(3, 15, C, C)).astype(np.float32), lengths=np.array([15, 8, 1], np.int32), B=3))
    check_path(dict(w=np.zeros((1, 6, C, C), np.float32), lengths=np.array([6], np.int32), B=1))
    # weights of up to about +-50 (all within the range the distance and the marginals are exact for)
    cfg = workloads.dense(B=2, T=14, V=V, order=1, sigma=12.0, seed=V)
    cfg["w"][rng.random(cfg["w"].shape) < 0.3] = -1.0e4
    cfg["w"][:, :, 2, :] = -1.0e4
    check_path(cfg)
    check_posteriors(cfg)
    cfg = workloads.dense(B=2, T=10, V=V, order=1, sigma=2.0, seed=V + 1)
    cfg["w"][rng.random(cfg["w"].shape) < 0.3] = -np.inf
    cfg["w"][:, 1:, 0, :] = np.finfo(np.float32).min           # the start state may not be left after the first frame
    check_posteriors(cfg)
    check_path(cfg)
    # no path at all: the distance is -inf and no marginal is anything but 0
    cfg["w"][:, 4] = -np.inf
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    D, g = lb.last_arc_posteriors(w, lengths)
    assert torch.all(D == -np.inf) and torch.all(g == 0)
    assert torch.all(lb.last_shortest_distance(w, lengths) == -np.inf)
    # far beyond scaled float32: right distance, and either right marginals or status 6
    cfg = workloads.dense(B=2, T=11, V=V, order=1, sigma=40.0, seed=4000 + V)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(w, lengths, item_status=status)
    assert_dist_close(D.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 1)[1])
    go = oracle.posteriors(cfg["w"], cfg["lengths"], 1)
    assert not torch.isnan(g).any()
    for b in range(2):
        assert int(status[b]) in (0, 6)
        if int(status[b]) == 0:
            assert np.max(np.abs(g[b].cpu().numpy() - go[b])) <= TOL_POST_ABS


@pytest.mark.parametrize("V", [1, 2, 3])
def test_fewest_states_have_no_range_limit(V):
    announce("bigram of fewer than five states, weights of up to +-180: right marginals, status 0, V", V)
    cfg = workloads.dense(B=3, T=12, V=V, order=1, sigma=40.0, seed=4000 + V, len_lo=9, len_hi=12)
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    status = torch.full((3,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(w, lengths, item_status=status)
    assert status.cpu().tolist() == [0, 0, 0]
    assert_dist_close(D.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 1)[1])
    # float32 scores of a few hundred in base 2 resolve 1.5e-5: a handful of roundings in an exponent
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(cfg["w"], cfg["lengths"], 1))) <= 5.0e-5
    assert_dist_close(lb.last_shortest_distance(w, lengths).cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 1)[1])


@pytest.mark.parametrize("V", [8, 32, 59, 95])
def test_marginals_beyond_the_range_stay_finite(V):
    announce("small bigram: a frame that only an arc of a vanished state can leave, V", V)
    C = V + 1
    w = np.zeros((1, 4, C, C), np.float32)
    w[0, 1:3] = -1000.0
    w[0, 1, :, 1] = 0.0                      # every state leads to state 1: its forward weight is the sum of C others
    w[0, 2, 1, 2] = 0.0                      # from there only to state 2,
    w[0, 3, 2] = -500.0                      # whose backward weight is far below the smallest float
    wd, lengths = dev(w), torch.tensor([4], dtype=torch.int32, device="cuda")
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(wd, lengths, item_status=status)
    assert_dist_close(D.cpu().numpy(), oracle.forward(w, np.array([4], np.int32), 1)[1])
    assert torch.isfinite(g).all() and int(status[0]) in (0, 6)
    base = torch.full_like(wd, 0.25)
    lb.last_arc_posteriors(wd, lengths, dw=base, scale=1.0, accumulate=True)
    assert torch.isfinite(base).all()


@pytest.mark.parametrize("V", [3, 4])
def test_more_frames_than_a_grid_has_rows(V):
    announce("small bigram: 66000 frames, V", V)
    T, C = 66000, V + 1
    w = np.full((1, T, C, C), -np.inf, np.float32)
    w[:, :, 0, 0] = 0.0                      # up to the last 60 frames only the empty label: nothing is rounded there
    w[:, -60:] = np.random.default_rng(V).normal(size=(1, 60, C, C))
    lengths = np.array([T], np.int32)
    D, g = lb.last_arc_posteriors(dev(w), dev(lengths))
    assert_dist_close(D.cpu().numpy(), oracle.forward(w, lengths, 1)[1])
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 1))) <= TOL_POST_ABS


def far_apart(kind, V, B=12, T=24):
    """weights whose differences within a row, between rows or between columns leave scaled float32"""
    C = V + 1
    rng = np.random.default_rng(1000 * V + len(kind))
    w = rng.normal(size=(B, T, C, C)).astype(np.float32)
    if kind == "one way up, the others later":
        # all but the way through state 1 fall behind by 2R, and make up for it in the next frame
        for b, R in enumerate([30, 40, 50, 60, 80, 200] * (B // 6)):
            p = [0, 3, 11, 12, 17, 22][b % 6]
            w[b, p], w[b, p + 1] = -R, R
            w[b, p, :, 1], w[b, p + 1, 1] = R, -R
    elif kind == "sigma 60":
        w *= 60.0
    elif kind == "rows and columns":
        w += 60.0 * rng.normal(size=(B, T, C, 1)).astype(np.float32) + 60.0 * rng.normal(size=(B, T, 1, C)).astype(np.float32)
    elif kind == "a column of -100":
        w[:, :, :, 1] = -100.0
        w[:, T // 2, 2:, :] = -300.0
    elif kind == "rows of -200":
        w[:, :, 1:3] = -200.0
        w[:, T // 3:T // 3 + 2, :, 3:] = -250.0
    lengths = np.full(B, T, np.int32)
    lengths[::4] = rng.integers(2, T, size=len(lengths[::4]))
    return w, lengths


@pytest.mark.parametrize("V", [4, 33, 60, 95])
@pytest.mark.parametrize("kind", ["one way up, the others later", "sigma 60", "rows and columns", "a column of -100",
                                  "rows of -200"])
def test_weights_far_apart(kind, V):
    announce("small bigram: right distances without marginals; with them right ones or status 6:", kind, V)
    w, lengths = far_apart(kind, V)
    wd, ld = dev(w), dev(lengths)
    B = len(lengths)
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    _, D_o = oracle.forward(w, lengths, 1)
    assert_dist_close(lb.last_shortest_distance(wd, ld, item_status=status).cpu().numpy(), D_o)
    assert status.cpu().tolist() == [0] * B
    D, g = lb.last_arc_posteriors(wd, ld, item_status=status)
    g_o = oracle.posteriors(w, lengths, 1)
    assert torch.isfinite(g).all()
    # (scores of a thousand: their float32 roundings are 3e-5 in an exponent)
    for b in range(B):
        assert int(status[b]) in (0, 6)
        if int(status[b]) == 0:
            assert_dist_close(D[b:b + 1].cpu().numpy(), D_o[b:b + 1])
            assert np.max(np.abs(g[b].cpu().numpy() - g_o[b])) <= 5.0e-5
