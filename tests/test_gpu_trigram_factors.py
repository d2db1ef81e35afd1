"""The trigram recursions whose sums are products of exponentials formed ahead of the chain (trigram_kernels.hpp), where those products
do not hold: weights of a column or row so far apart, or states so far behind, that a sum falls below 2^-60, so that the
workgroup takes the logarithms.  Against the float64 oracle; distances 1e-5 relative."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, assert_dist_close, dev

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
