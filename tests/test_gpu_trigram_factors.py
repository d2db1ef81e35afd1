"""The trigram recursions whose sums are products of exponentials formed ahead of the chain (trigram_kernels.hpp), where those products
do not hold: weights of a column or row so far apart, or states so far behind, that a sum falls below 2^-92, so that the
wave takes the logarithms.  Against the float64 oracle; distances 1e-5 relative."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, assert_dist_close, dev, library_option

pytestmark = pytest.mark.gpu


# 11, 12: one workgroup, two; 19, 20, 35, 36, 43: the edges of the instantiations; 44: none ahead
@pytest.mark.parametrize("V", [4, 11, 12, 17, 19, 20, 32, 35, 36, 43, 44])
@pytest.mark.parametrize("kind", ["columns", "rows", "frames", "one way", "missing"])
def test_weights_far_apart(kind, V):
    announce("trigram factors: weights far apart:", kind, V)
    rng = np.random.default_rng(V + 100 * len(kind))
    B, T, C = 3, 9, workloads.num_states(V, 2)
    w = rng.normal(size=(B, T, C, V + 1)).astype(np.float32)
    if kind == "columns":                                    # the largest weight of a column starts where nothing is
        w += rng.uniform(-120.0, 120.0, size=(B, T, C, V + 1)).astype(np.float32)
    elif kind == "rows":
        w += rng.uniform(-150.0, 150.0, size=(B, T, C, 1)).astype(np.float32)
    elif kind == "frames":
        w += rng.uniform(-300.0, 300.0, size=(B, T, 1, 1)).astype(np.float32)
    elif kind == "one way":                                  # all but one label fall behind and make up for it later
        w[:, 2:5, :, 1:V] -= 100.0
        w[:, 5:8, 1 + (V - 1):, :] += 90.0
    elif kind == "missing":
        w[rng.random(w.shape) < 0.5] = -np.inf
        w[:, 3, :, 1] = -np.inf
        w[:, 5, 1:1 + V // 2] = -1.0e4
    lengths = np.array([T, T - 1, 4], np.int32)
    wd, ld = dev(w), dev(lengths)
    D, g = lb.last_arc_posteriors(wd, ld, order=2)
    lb.check_item_status()
    _, D_o = oracle.forward(w, lengths, 2)
    g_o = oracle.posteriors(w, lengths, 2)
    assert_dist_close(D.cpu().numpy(), D_o)
    assert_dist_close(lb.last_shortest_distance(wd, ld, order=2).cpu().numpy(), D_o)
    # an exponent is a sum of scores of the size of `most`, each rounded to 2^-24 of it: a handful of such errors
    most = max(16.0, float(np.max(np.abs(np.where(np.isfinite(w) & (np.abs(w) < 9.0e3), w, 0.0)))))
    assert np.max(np.abs(g.cpu().numpy() - g_o)) <= max(1.0e-5, 8.0 * T * most * 2.0 ** -24)


@pytest.mark.parametrize("V", [12, 20, 36])
@pytest.mark.parametrize("sigma", [1.0, 3.0, 5.0, 10.0])
def test_as_precise_as_sums_of_differences(sigma, V):
    """Marginals where both factors have large arguments: no further from the oracle than those of the general kernel, which takes the
    exponential of each score's distance from the largest, and to neither side of it."""
    announce("trigram factors: precision:", sigma, V)
    B, T, C = 8, 24, workloads.num_states(V, 2)
    errors, sides = [], []
    for seed in range(2 if V == 36 else 4):
        cfg = workloads.dense(B=B, T=T, V=V, order=2, sigma=sigma, seed=10 * V + seed, C=C)
        want = torch.from_numpy(np.asarray(oracle.posteriors(cfg["w"], cfg["lengths"], 2))).cuda()
        w, lengths = dev(cfg["w"]), dev(cfg["lengths"])

        def far():
            off = lb.last_arc_posteriors(w, lengths, order=2)[1].double() - want
            side = off.sum((1, 2, 3)) / want.sum((1, 2, 3))
            return (off.flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).mean().item(), side.mean().item()
        new = far()
        with library_option(lb.OPT_FORCE_SOLO, 1):
            old = far()
        errors.append((new[0], old[0]))
        sides.append(new[1])
    (new, old), side = np.mean(errors, axis=0), np.mean(sides)
    print("error %.2e / %.2e, mean of the signed errors %+.1e" % (new, old, side), flush=True)
    assert new <= 0.9 * old
    # roundings go both ways; a constant that is off (log2 e by 1.3e-8 of itself, for arguments of some 2 sigma) does not
    assert abs(side) <= 1.0e-7


@pytest.mark.parametrize("V", [4, 12, 20, 33, 36, 43])
@pytest.mark.parametrize("mask", [-7.1e5, -1.0e9, -1.0e10, -3.0e38, float(np.finfo(np.float32).min), -np.inf])
def test_masks_as_largest_weights(mask, V):
    """Labels that nothing may emit and histories that nothing may leave: the largest weight of a column or of a row is the mask."""
    announce("trigram factors: masks:", mask, V)
    rng = np.random.default_rng(V)
    B, T, C = 3, 9, workloads.num_states(V, 2)
    w = rng.normal(size=(B, T, C, V + 1)).astype(np.float32)
    w[:, :, :, V // 2 + 1] = mask                                    # a label
    w[:, 1:, 1 + V:1 + V + V // 2] = mask                            # histories (1, 1) to (1, V / 2)
    w[0, 4, :, 1 + V // 3] = mask                                    # a label in one frame
    w[1, 3, 2] = mask
    lengths = np.array([T, T - 1, 4], np.int32)
    wd, ld = dev(w), dev(lengths)
    D, g = lb.last_arc_posteriors(wd, ld, order=2)
    lb.check_item_status()
    _, D_o = oracle.forward(w, lengths, 2)
    assert_dist_close(D.cpu().numpy(), D_o)
    assert_dist_close(lb.last_shortest_distance(wd, ld, order=2).cpu().numpy(), D_o)
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 2))) <= 1.0e-5


@pytest.mark.parametrize("level", [-3.0e38, -1.0e10, -1.0e9, -6.0e5, 6.0e5, 1.0e9, 2.0e9, 1.0e30])
@pytest.mark.parametrize("V", [12, 20, 36])
def test_levels_of_frames(V, level):
    """One frame all of whose weights are far from the others': the distance is still the sum of both."""
    announce("trigram factors: levels:", level, V)
    rng = np.random.default_rng(V)
    B, T, C = 2, 7, workloads.num_states(V, 2)
    w = rng.normal(size=(B, T, C, V + 1)).astype(np.float32)
    w[:, 3] += np.float32(level)
    lengths = np.array([T, T - 2], np.int32)
    wd, ld = dev(w), dev(lengths)
    D, g = lb.last_arc_posteriors(wd, ld, order=2)
    lb.check_item_status()
    _, D_o = oracle.forward(w, lengths, 2)
    assert_dist_close(D.cpu().numpy(), D_o)
    assert_dist_close(lb.last_shortest_distance(wd, ld, order=2).cpu().numpy(), D_o)
    assert not np.isnan(g.cpu().numpy()).any()


# the largest weights of a column belong to histories that no path is in: at the item's start, and where nothing may lead there
@pytest.mark.parametrize("V", [4, 12, 17, 20, 35, 36, 43])
@pytest.mark.parametrize("kind", ["start", "label"])
def test_large_weights_of_histories_that_no_path_is_in(kind, V):
    announce("trigram factors: weights of histories that no path is in:", kind, V)
    rng = np.random.default_rng(V)
    B, T, C = 3, 9, workloads.num_states(V, 2)
    w = rng.normal(size=(B, T, C, V + 1)).astype(np.float32)
    if kind == "start":                                      # one label after one frame, two after two
        w[:, 1, :1 + V] -= 150.0
        w[:, 1, 1 + V:] += 150.0
    else:                                                    # histories (a, b) are 1 + V + (a - 1) V + b - 1
        y = V // 2
        w[:, :, :, y] = -np.inf
        w[:, :, 1 + V:] -= 100.0
        w[:, :, 1 + V + (y - 1) * V:1 + V + y * V] += 300.0
        w[:, 3, 1 + V + (y - 1) * V] = 600.0
    lengths = np.array([T, T - 1, 4], np.int32)
    wd, ld = dev(w), dev(lengths)
    D, g = lb.last_arc_posteriors(wd, ld, order=2)
    lb.check_item_status()
    _, D_o = oracle.forward(w, lengths, 2)
    assert_dist_close(D.cpu().numpy(), D_o)
    assert_dist_close(lb.last_shortest_distance(wd, ld, order=2).cpu().numpy(), D_o)
    # scores of up to 300 T (one is 600), each rounded to 2^-24 of it
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 2))) <= 8.0 * T * 300.0 * 2.0 ** -24
