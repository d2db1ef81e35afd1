"""Marginals and distances of the kernels for small dense frames (bigram_kernels.hpp, trigram_kernels.hpp,
table_chain_kernels.hpp, marginals_kernels.hpp) are as close to the float64 oracle as those of the general kernels
that the library options select."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, dev, library_option
from test_gpu_tables_local import both_orders

pytestmark = pytest.mark.gpu


def errors(cfg, w, lengths, g_order, want, D_o):
    """relative error of all marginals of an item together, and of the distances, averaged over the items"""
    D, g = lb.last_arc_posteriors(w, lengths, order=g_order)
    far = (g.double() - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)
    d1 = np.abs(D.double().cpu().numpy() - D_o) / np.abs(D_o)
    d2 = np.abs(lb.last_shortest_distance(w, lengths, order=g_order).double().cpu().numpy() - D_o) / np.abs(D_o)
    return far.mean().item(), d1.mean(), d2.mean()


# order, labels, states of a table, items; the option that selects the general kernels
@pytest.mark.parametrize("order,V,C,B", [(1, 2, 0, 64), (1, 4, 0, 64), (1, 32, 0, 16), (1, 80, 0, 8), (2, 3, 0, 64), (2, 20, 0, 4),
                                         (0, 12, 200, 16), (0, 40, 6, 64)])
@pytest.mark.parametrize("sigma", [1.5, 12.0])
def test_as_precise_as_the_general_kernels(order, V, C, B, sigma):
    announce("precision: order, V, C, sigma", order, V, C, sigma)
    if order:
        C = workloads.num_states(V, order)
    cfg = workloads.dense(B=B, T=61, V=V, order=order or 1, sigma=sigma, seed=1000 + V, C=C)
    o_order, g_order = both_orders(workloads.random_table(C, V, seed=C)) if order == 0 else (order, order)
    _, D_o = oracle.forward(cfg["w"], cfg["lengths"], o_order)
    want = torch.from_numpy(np.asarray(oracle.posteriors(cfg["w"], cfg["lengths"], o_order))).cuda()
    w, lengths = dev(cfg["w"]), dev(cfg["lengths"])
    new = errors(cfg, w, lengths, g_order, want, D_o)
    option = (lb.OPT_CLUSTER_GENERATION, 2) if order == 1 and C >= 5 else (lb.OPT_FORCE_SOLO, 1)
    with library_option(*option):
        old = errors(cfg, w, lengths, g_order, want, D_o)
    print("marginals %.2e / %.2e, distances %.2e / %.2e, %.2e / %.2e" % (new[0], old[0], new[1], old[1], new[2], old[2]), flush=True)
    assert new[0] <= 0.9 * old[0]
    # (a distance is a float32 number, whose own rounding is most of either error)
    assert new[1] <= 1.05 * old[1] and new[2] <= 1.05 * old[2]
