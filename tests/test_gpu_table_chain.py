"""Table contexts whose frame the threads of one workgroup own (table_chain_kernels.hpp), at the edges of
its instantiations and with arcs crowded into few states, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import brute_force as bf
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev, library_option
from test_gpu_tables_local import both_orders, check_table_lattice

pytestmark = pytest.mark.gpu


# C (V + 1) arcs a frame: 4 the fewest, 4096/4100, 8190, 8192/8196 the edges of the instantiations, 16384 the most
# taken and 16388 the first left to the older kernels; ends that are no multiple of four; 61 arcs a row
@pytest.mark.parametrize("C,V", [(2, 1), (1, 3), (1, 4), (512, 7), (205, 19), (819, 9), (1024, 7), (683, 11), (270, 60),
                                 (4096, 3), (4097, 3)])
def test_sizes(C, V):
    announce("table chain, C, V", C, V)
    cfg = workloads.dense(B=4, T=7, V=V, sigma=1.5, seed=C + V, C=C)
    cfg["lengths"] = np.array([7, 0, 1, 4], np.int32)
    cfg["w"][2, 1:] = np.nan
    table = workloads.random_table(C, V, seed=C)
    check_table_lattice(cfg, table)


@pytest.mark.parametrize("C,V", [(40, 25), (300, 9)])
def test_crowded_destinations_missing_arcs_and_older_kernels(C, V):
    announce("table chain: all arcs into one state, -inf and -1e4 arcs; one workgroup per item, C, V", C, V)
    rng = np.random.default_rng(C)
    cfg = workloads.dense(B=2, T=9, V=V, sigma=2.0, seed=C, C=C)
    check_table_lattice(cfg, np.full((C, V), C - 1, np.int32))
    table = workloads.random_table(C, V, seed=C)
    cfg["w"][rng.random(cfg["w"].shape) < 0.2] = -np.inf
    cfg["w"][rng.random(cfg["w"].shape) < 0.2] = -1.0e4
    cfg["w"][:, :, 0, 0] = 0.0                                 # a path is left
    check_table_lattice(cfg, table)
    with library_option(lb.OPT_FORCE_SOLO, 1):
        check_table_lattice(cfg, table)
    # more items than compute units
    many = workloads.dense(B=300, T=5, V=V, sigma=1.0, seed=C, len_lo=0, len_hi=5, C=C)
    check_table_lattice(many, table)


def test_bad_table_is_reported_by_every_call():
    announce("table chain: an entry that names no state")
    table = workloads.random_table(30, 6, seed=2)
    table[4, 2] = 30
    _, g0 = both_orders(np.minimum(table, 29))
    g0 = dev(table)
    w, lengths = torch.zeros((2, 5, 30, 7), device="cuda"), dev(np.array([5, 3], np.int32))
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(w, lengths, order=g0, item_status=status)
    assert status.cpu().tolist() == [7, 7] and torch.isnan(D).all() and not torch.isinf(g).any()
    assert torch.isnan(lb.last_shortest_distance(w, lengths, order=g0, item_status=status)).all()
    assert status.cpu().tolist() == [7, 7]
    labels, _, score = lb.last_shortest_path(w, lengths, order=g0, item_status=status)
    assert status.cpu().tolist() == [7, 7] and torch.isnan(score).all() and torch.all(labels == -1)


@pytest.mark.parametrize("V", [2, 5])
def test_weights_of_unreachable_states_do_not_matter(V):
    announce("table chain: NaN and +inf on arcs out of states that no path has reached yet, V", V)
    table, _ = bf.history_table(V, 3)
    C = table.shape[0]
    cfg = workloads.dense(B=2, T=9, V=V, sigma=1.0, seed=V, len_lo=6, len_hi=9, C=C)
    o0, g0 = both_orders(table)
    lengths = dev(cfg["lengths"])
    _, D_o = oracle.forward(cfg["w"], cfg["lengths"], o0)
    g_o = oracle.posteriors(cfg["w"], cfg["lengths"], o0)
    cfg["w"][:, 0, 1:] = np.nan                                # only the start state
    cfg["w"][:, 1, 1 + V:, ::2] = np.inf                       # histories of at most one label
    cfg["w"][:, 1, 1 + V:, 1::2] = np.nan
    w = dev(cfg["w"])
    for solo in (0, 1):
        with library_option(lb.OPT_FORCE_SOLO, solo):
            D, g = lb.last_arc_posteriors(w, lengths, order=g0)
            assert_dist_close(D.cpu().numpy(), D_o)
            assert np.max(np.abs(g.cpu().numpy() - g_o)) <= TOL_POST_ABS
