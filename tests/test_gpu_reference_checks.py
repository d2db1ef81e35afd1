"""The check of the reference strings (contexts, chains of positions with equal context) and the rows of the locally normalised
gradient at the edges of their kernels, against the float64 oracle with the tolerances of test_gpu_parity."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, dev

pytestmark = pytest.mark.gpu


# 64 positions are compared at a time; with two labels nearly all positions are in a chain with others
@pytest.mark.parametrize("V,U", [(2, 63), (2, 64), (2, 65), (3, 129), (40, 130), (140, 70)])
def test_chains_of_equal_contexts(V, U):
    announce("reference check: labels, reference length", V, U)
    rng = np.random.default_rng(V * 1000 + U)
    B, T, C = 4, U + 9, V + 1
    w = rng.normal(size=(B, T, C, C)).astype(np.float32)
    lengths = np.array([T, T - 3, U, T], np.int32)
    refs = rng.integers(1, V + 1, size=(B, U)).astype(np.int32)
    refs[3] = 1 + np.arange(U) % V
    ulen = np.array([U, U - 1, U, 1], np.int32)
    wd, ld, rd, ud = dev(w), dev(lengths), dev(refs), dev(ulen)
    table = np.tile(np.arange(1, C, dtype=np.int32), (C, 1))
    o = oracle.numerator_local(w, lengths, refs, ulen, 1)
    n = oracle.numerator(w, lengths, refs, ulen, 1)
    for order in (1, dev(table)):
        base = torch.full_like(wd, 0.25)
        for g, add in ((torch.full_like(wd, 7.0), False), (base, True)):
            ll = lb.last_local_log_likelihood(wd, ld, rd, ud, order=order, dw=g, accumulate=add)
            lb.check_item_status()
            assert np.max(np.abs(ll.cpu().numpy() - o["N"]) / np.maximum(1, np.abs(o["N"]))) < 1e-5
            assert np.max(np.abs(g.cpu().numpy() - (0.25 if add else 0.0) - o["grad"])) < 1e-5
        num = lb.last_intersect_reference(wd, ld, rd, ud, order=order)
        assert np.max(np.abs(num.cpu().numpy() - n["N"]) / np.maximum(1, np.abs(n["N"]))) < 1e-5


@pytest.mark.parametrize("C,V", [(300, 40), (301, 40), (2000, 9)])
def test_tables_in_and_out_of_lds(C, V):
    announce("reference check: table of states, labels", C, V)
    rng = np.random.default_rng(C)
    B, T, U = 2, 24, 15
    table = workloads.random_table(C, V, 5)
    w = rng.normal(size=(B, T, C, V + 1)).astype(np.float32)
    lengths, ulen = np.array([T, 20], np.int32), np.array([U, 11], np.int32)
    refs = rng.integers(1, V + 1, size=(B, U)).astype(np.int32)
    oracle.set_next_table(table)
    o = oracle.numerator_local(w, lengths, refs, ulen, 0)
    g = torch.empty_like(dev(w))
    ll = lb.last_local_log_likelihood(dev(w), dev(lengths), dev(refs), dev(ulen), order=dev(table), dw=g)
    lb.check_item_status()
    assert np.max(np.abs(ll.cpu().numpy() - o["N"]) / np.maximum(1, np.abs(o["N"]))) < 1e-5
    assert np.max(np.abs(g.cpu().numpy() - o["grad"])) < 1e-5


# beside the clusters of a denominator the check runs on two waves for references of up to 512 labels
@pytest.mark.parametrize("U", [1, 130, 512, 513])
def test_check_beside_a_clustered_denominator(U):
    announce("reference check beside a clustered denominator: labels, reference length", 100, U)
    rng = np.random.default_rng(U)
    B, T, V = 2, U + 4, 100
    w = rng.normal(size=(B, T, V + 1, V + 1)).astype(np.float32)
    refs = rng.integers(1, V + 1, size=(B, U)).astype(np.int32)
    refs[1, ::2] = 7
    args = dev(w), dev(np.array([T, T - 2], np.int32)), dev(refs), dev(np.array([U, max(U - 3, 0)], np.int32))
    _, N, g = lb.last_globally_normalized_loss(*args, order=1)
    lb.check_item_status()
    g2 = torch.empty_like(g)
    lb.last_arc_posteriors(*args[:2], order=1, dw=g2)
    assert torch.equal(N, lb.last_intersect_reference(*args, order=1, dw=g2, scale=-1.0, accumulate=True))
    assert float((g - g2).abs().max()) < 2e-5
