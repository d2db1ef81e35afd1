"""The chain of small bigrams in one wavefront (bigram_wave_kernels.hpp) against the float64 oracle where it can go wrong:
label counts at the edges of its tiles and of their instantiations, lengths around its groups of 4 and 8 frames, frames
whose scale the bound from the frame before misses.  Tolerances of test_gpu_parity."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, assert_dist_close, dev
from test_gpu_parity import check_path, check_posteriors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4, 5, 8, 9, 16, 17, 18, 33, 35, 49, 50])
def test_groups_of_frames(V):
    announce("one-wave bigram, lengths around its groups, V", V)
    T = 34
    cfg = workloads.dense(B=12, T=T, V=V, order=1, sigma=2.0, seed=500 + V)
    cfg["lengths"] = np.array([1, 4, 5, 7, 15, 16, 17, 23, 24, 31, 33, 34], np.int32)
    check_posteriors(cfg)
    check_path(cfg)
    dist = lb.last_shortest_distance(dev(cfg["w"]), dev(cfg["lengths"]))
    assert_dist_close(dist.cpu().numpy(), oracle.forward(cfg["w"], cfg["lengths"], 1)[1])


@pytest.mark.parametrize("V", [7, 32, 48, 64])
def test_scales_that_no_bound_foresees(V):
    announce("one-wave bigram, rows of a frame up to 2^70 apart, frames up to 2^200 apart, V", V)
    rng = np.random.default_rng(V)
    B, T, C = 6, 21, V + 1
    w = rng.normal(size=(B, T, C, C)).astype(np.float32)
    w += rng.uniform(-60.0, 60.0, size=(B, T, 1, 1)).astype(np.float32)              # frames
    w[:3] += rng.uniform(-20.0, 20.0, size=(3, T, C, 1)).astype(np.float32)          # rows
    w[3:, :, :, 1:V // 2] -= rng.uniform(0.0, 25.0, size=(3, T, 1, 1)).astype(np.float32)    # columns
    w[1, ::3, 0] += 30.0                                                             # the start state's row alone
    lengths = np.array([21, 20, 19, 21, 18, 17], np.int32)
    wd, ld = dev(w), dev(lengths)
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(wd, ld, item_status=status)
    _, D_o = oracle.forward(w, lengths, 1)
    assert status.cpu().tolist() == [0] * B
    assert_dist_close(D.cpu().numpy(), D_o)
    # (scores of up to a thousand: their float32 roundings are 3e-5 in an exponent)
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 1))) <= 5.0e-5
    assert_dist_close(lb.last_shortest_distance(wd, ld, item_status=status).cpu().numpy(), D_o)
    check_path(dict(w=w, lengths=lengths, B=B))


@pytest.mark.parametrize("V", [3, 6, 31, 47, 64])
def test_paths_of_many_segments(V):
    announce("one-wave bigram, paths over more frames than one pass of the backpointer kernel, V", V)
    rng = np.random.default_rng(10 + V)
    T, C = 1300, V + 1                                     # segments of 37 frames, the kernel takes 32 at a time
    w = rng.integers(-2, 3, size=(2, T, C, C)).astype(np.float32)          # (ties everywhere)
    w[rng.random(w.shape) < 0.2] = -np.inf
    check_path(dict(w=w, lengths=np.array([T, 1111], np.int32), B=2))


@pytest.mark.parametrize("V", [3, 8, 31, 48, 64])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_paths_past_weights_that_count_nowhere(V, value):
    announce("one-wave bigram, paths, weights of states that no path is in: V, value", V, value)
    rng = np.random.default_rng(V)
    B, T, C = 3, 41, V + 1
    for kind in range(3):
        w = rng.normal(size=(B, T, C, C)).astype(np.float32)
        if kind == 2:
            w[:, 0, 0, 0] = -np.inf                          # the start state is left at once
        nowhere = w[:, 1:, 0] if kind == 2 else w[:, 0, 1:]
        lengths = np.array([T, T - 1, 7], np.int32)
        want = oracle.viterbi(w, lengths, 1, "f32")
        nowhere[rng.random(nowhere.shape) < (0.4 if kind == 0 else 1.0)] = value
        got = lb.last_shortest_path(dev(w), dev(lengths))
        for g, x in zip(got, want):
            assert np.array_equal(g.cpu().numpy(), x)


@pytest.mark.parametrize("V", [4, 9, 32, 47, 64])
def test_distance_of_weights_that_are_no_number(V):
    announce("one-wave bigram, distance, NaN on the arcs of a state that is left: V", V)
    rng = np.random.default_rng(V)
    B, T, C = 3, 31, V + 1
    w = rng.normal(size=(B, T, C, C)).astype(np.float32)
    w[:2, 0, 0, 0] = -np.inf
    w[:2, 1:, 0] = np.nan
    lengths = np.array([T, T - 1, T], np.int32)
    got = lb.last_shortest_distance(dev(w), dev(lengths)).cpu().numpy()
    assert np.isnan(got[:2]).all()                           # (0 times NaN: never a number that looks like a distance)
    assert_dist_close(got[2:], oracle.forward(w[2:], lengths[2:], 1)[1])


# (labels, most items on one wave) of paths, best scores and distances: both sides of where other kernels take over
@pytest.mark.parametrize("call,V,B", [("path", 3, 256), ("path", 16, 256), ("path", 20, 256), ("path", 31, 214), ("path", 32, 202), ("path", 47, 95),
                                      ("path", 48, 91), ("path", 63, 53), ("path", 64, 192), ("score", 33, 256), ("score", 63, 256),
                                      ("distance", 4, 256), ("distance", 16, 256), ("distance", 17, 128), ("distance", 31, 128),
                                      ("distance", 33, 512), ("distance", 56, 512), ("distance", 57, 192), ("distance", 63, 192)])
def test_batches_on_both_sides_of_the_rule(call, V, B):
    announce("one-wave bigram and more items than it is taken for:", call, V, B)
    rng = np.random.default_rng(V)
    T, C = 9, V + 1
    w = rng.normal(size=(B + 1, T, C, C)).astype(np.float32)
    w[::2] = np.round(w[::2])                                # (ties)
    w[rng.random(w.shape) < 0.1] = -np.inf
    lengths = rng.integers(0, T + 1, size=B + 1).astype(np.int32)
    for n in (B, B + 1):
        wd, ld = dev(w[:n]), dev(lengths[:n])
        if call == "path":
            for g, x in zip(lb.last_shortest_path(wd, ld), oracle.viterbi(w[:n], lengths[:n], 1, "f32")):
                assert np.array_equal(g.cpu().numpy(), x)
        elif call == "score":
            got = lb.last_shortest_distance(wd, ld, semiring="tropical")
            assert np.array_equal(got.cpu().numpy(), oracle.viterbi(w[:n], lengths[:n], 1, "f32")[2])
        else:
            assert_dist_close(lb.last_shortest_distance(wd, ld).cpu().numpy(), oracle.forward(w[:n], lengths[:n], 1)[1])
