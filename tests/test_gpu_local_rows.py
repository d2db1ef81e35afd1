"""The locally normalised log-likelihood and its gradient over the row lengths and context sets at which the
kernels' pieces change, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import TOL_POST_ABS, announce, assert_dist_close, dev

pytestmark = pytest.mark.gpu


# V + 1 floats a row: 3 (no 16-byte piece), 4, 5, 256/257 (one or two pieces a lane), 512/513 (two, or a loop);
# order 2 with 33 931 states: more than the marks of a frame hold, the tensor is filled by another kernel
@pytest.mark.parametrize("V,order,T,U", [(2, 1, 9, 4), (3, 1, 9, 6), (4, 1, 9, 5), (255, 1, 7, 5), (256, 1, 7, 6),
                                         (511, 1, 6, 4), (512, 1, 6, 4), (184, 2, 3, 2), (9, 2, 12, 7)])
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
