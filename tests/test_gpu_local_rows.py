"""The locally normalised log-likelihood and its gradient over the row lengths and context sets at which the
kernels' pieces change, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev
from test_gpu_tables_local import both_orders

pytestmark = pytest.mark.gpu


# V + 1 floats a row: 3 (no 16-byte piece), 4, 5, 256/257 (one or two pieces a lane), 512/513 (two, or a loop), 800
# (frames of 2.5 MB, several workgroups each);
# order 2 with 33 931 states: more than the marks of a frame hold, the tensor is filled by another kernel
@pytest.mark.parametrize("V,order,T,U", [(2, 1, 9, 4), (3, 1, 9, 6), (4, 1, 9, 5), (255, 1, 7, 5), (256, 1, 7, 6),
                                         (511, 1, 6, 4), (512, 1, 6, 4), (799, 1, 5, 4), (184, 2, 3, 2), (9, 2, 12, 7)])
def test_rows(V, order, T, U):
    announce("local rows: V, order, T, U", V, order, T, U)
    cfg = workloads.config(3, B=4 if order == 1 or V < 100 else 1, T=T, V=V, order=order, Umax=U, u_lo=1, u_hi=U)
    B = cfg["B"]
    cfg["lengths"] = np.array([T, T - 1, T, 2][:B], np.int32)
    cfg["ref_lengths"] = np.array([U, 1, 0, 2][:B], np.int32)
    cfg["w"][np.random.default_rng(V).random(cfg["w"].shape) < 0.1] = -1.0e4
    w, lengths, refs, ulen = (dev(cfg[k]) for k in ("w", "lengths", "refs", "ref_lengths"))
    lo = oracle.numerator_local(cfg["w"], cfg["lengths"], cfg["refs"], cfg["ref_lengths"], order)
    g = torch.full_like(w, 7.0)
    ll = lb.last_local_log_likelihood(w, lengths, refs, ulen, order=order, dw=g)
    assert_dist_close(ll.cpu().numpy(), lo["N"])
    assert np.max(np.abs(g.cpu().numpy() - lo["grad"])) <= TOL_POST_ABS
    base = torch.full_like(w, 0.25)
    lb.last_local_log_likelihood(w, lengths, refs, ulen, order=order, dw=base, scale=-2.0, accumulate=True)
    assert torch.max(torch.abs(base - (0.25 - 2.0 * g))).item() < 1e-6


# rows of 513, 515, 1024, 1025 and 3000 weights, all cells of a frame in one or two chains
@pytest.mark.parametrize("V,C", [(512, 1), (514, 2), (1023, 1), (1024, 1), (2999, 2)])
def test_long_rows_and_chains(V, C):
    announce("local rows of more than 512 weights, long chains: V, C", V, C)
    T, U = 21, 12
    cfg = workloads.dense(B=3, T=T, V=V, sigma=1.5, seed=V, C=C)
    refs, ulen = workloads.references(np.random.default_rng(V), 3, V, U, 0, U)
    refs[0, 1::2] = refs[0, 0]                                  # one label several times
    cfg["lengths"] = np.array([T, T - 1, 13], np.int32)
    ulen[0] = U
    cfg["w"][np.random.default_rng(V).random(cfg["w"].shape) < 0.1] = -1.0e4
    o0, g0 = both_orders(workloads.random_table(C, V, seed=C))
    w, lengths, r, n = dev(cfg["w"]), dev(cfg["lengths"]), dev(refs), dev(ulen)
    lo = oracle.numerator_local(cfg["w"], cfg["lengths"], refs, ulen, o0)
    g = torch.full_like(w, 7.0)
    ll = lb.last_local_log_likelihood(w, lengths, r, n, order=g0, dw=g)
    assert_dist_close(ll.cpu().numpy(), lo["N"])
    assert np.max(np.abs(g.cpu().numpy() - lo["grad"])) <= TOL_POST_ABS
    base = torch.full_like(w, 0.25)
    lb.last_local_log_likelihood(w, lengths, r, n, order=g0, dw=base, scale=-2.0, accumulate=True)
    assert torch.max(torch.abs(base - (0.25 - 2.0 * g))).item() < 1e-6


# rows in order or zeros of a frame first: as many reference labels as rows, one fewer and one more; a frame's rows by several workgroups
# (300 labels); a tensor of 272 MB with references of a fifth of its rows, and of one label less
@pytest.mark.parametrize("B,T,V,U", [(3, 12, 3, 2), (3, 12, 3, 3), (3, 12, 3, 4), (2, 40, 32, 31), (2, 40, 32, 32), (2, 40, 32, 33),
                                     (1, 310, 300, 299), (1, 310, 300, 300), (2, 520, 255, 51), (2, 520, 255, 50)])
def test_order_of_rows(B, T, V, U):
    announce("local rows: in order or not: B, T, V, U", B, T, V, U)
    cfg = workloads.config(3, B=B, T=T, V=V, order=1, Umax=U, u_lo=1, u_hi=U)
    cfg["lengths"] = np.array([T, T - 1, T - 2][:B], np.int32)
    cfg["ref_lengths"] = np.array([U, U // 2, 0][:B], np.int32)
    w, lengths, refs, ulen = (dev(cfg[k]) for k in ("w", "lengths", "refs", "ref_lengths"))
    lo = oracle.numerator_local(cfg["w"], cfg["lengths"], cfg["refs"], cfg["ref_lengths"], 1)
    want = torch.from_numpy(lo["grad"]).cuda()
    g = torch.full_like(w, 7.0)
    ll = lb.last_local_log_likelihood(w, lengths, refs, ulen, order=1, dw=g)
    lb.check_item_status()
    assert_dist_close(ll.cpu().numpy(), lo["N"])
    assert torch.max(torch.abs(g - want)).item() <= TOL_POST_ABS
    base = torch.full_like(w, 0.25)
    lb.last_local_log_likelihood(w, lengths, refs, ulen, order=1, dw=base, accumulate=True)
    assert torch.max(torch.abs(base - 0.25 - want)).item() <= TOL_POST_ABS


# arcs that do not exist and masks: lowest values, and some whose product with log2 e leaves float32 or its whole numbers; rows of one or
# two pieces a lane, of more, and of less than one.  The weights of what the reference reads stay, so that the likelihood is finite.
@pytest.mark.parametrize("V", [3, 4, 255, 256, 511, 512, 799])
@pytest.mark.parametrize("mask", [-np.inf, float(np.finfo(np.float32).min), -1.0e30, -1.3e10])
def test_missing_and_masked_arcs(V, mask):
    announce("local rows: masked arcs: V, mask", V, mask)
    T, U = 7, 4
    cfg = workloads.config(3, B=3, T=T, V=V, order=1, Umax=U, u_lo=1, u_hi=U)
    cfg["lengths"] = np.array([T, T - 1, 5], np.int32)
    cfg["ref_lengths"] = np.array([U, 2, 0], np.int32)
    shape = cfg["w"].shape
    hide = np.random.default_rng(V).random(shape) < 0.4
    hide[:, :, :, 0] = False
    for b in range(3):
        for r in cfg["refs"][b]:
            hide[b, :, :, r] = False
    cfg["w"][hide] = mask
    unread = np.setdiff1d(np.arange(1, V + 1), cfg["refs"][0])
    if unread.size:
        cfg["w"][0, :, unread[0]] = mask                        # a row that no path visits has none at all
    w, lengths, refs, ulen = (dev(cfg[k]) for k in ("w", "lengths", "refs", "ref_lengths"))
    lo = oracle.numerator_local(cfg["w"], cfg["lengths"], cfg["refs"], cfg["ref_lengths"], 1)
    assert np.all(np.isfinite(lo["N"])) and np.all(np.isfinite(lo["grad"]))
    g = torch.full_like(w, 7.0)
    ll = lb.last_local_log_likelihood(w, lengths, refs, ulen, order=1, dw=g)
    lb.check_item_status()
    assert_dist_close(ll.cpu().numpy(), lo["N"])
    assert np.max(np.abs(g.cpu().numpy() - lo["grad"])) <= TOL_POST_ABS
    base = torch.full_like(w, 0.25)
    lb.last_local_log_likelihood(w, lengths, refs, ulen, order=1, dw=base, accumulate=True)
    assert np.max(np.abs(base.cpu().numpy() - 0.25 - lo["grad"])) <= TOL_POST_ABS
