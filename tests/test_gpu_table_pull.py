"""Table contexts on lists of arcs (table_pull_kernels.hpp) against the float64 oracle at the edges of what they take; tolerances of
test_gpu_parity."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev

pytestmark = pytest.mark.gpu


def check(w, lengths, table):
    oracle.set_next_table(table)
    wd, ld, td = dev(w), dev(lengths), dev(table)
    D, g = lb.last_arc_posteriors(wd, ld, order=td)
    lb.check_item_status()
    again, g2 = lb.last_arc_posteriors(wd, ld, order=td)
    assert torch.equal(D, again) and torch.equal(g, g2)              # (sums in the order of the arcs, whatever the timing)
    D_o = oracle.forward(w, lengths, 0)[1]
    assert_dist_close(D.cpu().numpy(), D_o)
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 0))) <= TOL_POST_ABS
    assert_dist_close(lb.last_shortest_distance(wd, ld, order=td).cpu().numpy(), D_o)


# arcs from 3072 (just taken) to 8192; one to sixteen lanes a row; 1024 states; odd numbers of frames; distances of T / 2 frames
@pytest.mark.parametrize("C,V,T", [(1024, 2, 97), (1023, 6, 50), (1024, 7, 49), (513, 5, 48), (512, 15, 48), (256, 11, 96),
                                   (130, 62, 49), (61, 60, 48), (50, 63, 50)])
def test_sizes(C, V, T):
    announce("table lists: states, labels, frames", C, V, T)
    rng = np.random.default_rng(C)
    w = (1.5 * rng.normal(size=(2, T, C, V + 1))).astype(np.float32)
    w[1, T - 3:] = np.nan                                            # frames past the length are not read into a result
    check(w, np.array([T, T - 3], np.int32), workloads.random_table(C, V, V))


def test_lopsided_tables_missing_arcs_and_jumps():
    announce("table lists: states with up to 3000 arcs, arcs that do not exist, frames far apart")
    C, V, T = 250, 14, 51
    rng = np.random.default_rng(3)
    table = workloads.random_table(C, V, 1)
    table[5:, 2:] = 7                                                # nearly all arcs lead to one state
    w = rng.normal(size=(3, T, C, V + 1)).astype(np.float32)
    w[1] += rng.uniform(-30.0, 30.0, size=(T, 1, 1)).astype(np.float32)
    w[2][rng.random(w[2].shape) < 0.6] = -np.inf
    lengths = np.array([T, T, T - 1], np.int32)
    oracle.set_next_table(table)
    wd, ld, td = dev(w), dev(lengths), dev(table)
    D, g = lb.last_arc_posteriors(wd, ld, order=td)
    lb.check_item_status()
    assert_dist_close(D.cpu().numpy(), oracle.forward(w, lengths, 0)[1])
    # (scores of up to 60 between frames: float32 roundings of 4e-6 in an exponent, a few of them)
    assert np.max(np.abs(g.cpu().numpy() - oracle.posteriors(w, lengths, 0))) <= 3.0e-5
    # an arc out of a state that cannot be reached does not count, whatever its weight
    stay = np.tile(np.arange(C, dtype=np.int32)[:, None], (1, V))
    stay[0, 0] = 1
    v = rng.normal(size=(1, T, C, V + 1)).astype(np.float32)
    oracle.set_next_table(stay)
    want = oracle.forward(v, np.array([T], np.int32), 0)[1]
    v[:, :, 2:] = np.inf
    got = lb.last_shortest_distance(dev(v), dev(np.array([T], np.int32)), order=dev(stay))
    D, _ = lb.last_arc_posteriors(dev(v), dev(np.array([T], np.int32)), order=dev(stay))
    assert_dist_close(D.cpu().numpy(), want)


def test_status_and_a_bad_table():
    announce("table lists: lengths 0, invalid; a table entry that names no state")
    C, V, T = 400, 8, 50
    w = np.random.default_rng(1).normal(size=(4, T, C, V + 1)).astype(np.float32)
    lengths = np.array([T, 0, T + 1, -1], np.int32)
    table = workloads.random_table(C, V, 2)
    status = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    D, g = lb.last_arc_posteriors(dev(w), dev(lengths), order=dev(table), item_status=status)
    assert status.cpu().tolist() == [0, 0, 1, 1]
    assert float(D[1]) == 0.0 and torch.isnan(D[2:]).all() and torch.all(g[1:] == 0)
    table[3, 3] = C
    D, g = lb.last_arc_posteriors(dev(w), dev(lengths), order=dev(table), item_status=status)
    assert status.cpu().tolist() == [7] * 4 and torch.isnan(D).all()
