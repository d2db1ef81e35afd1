"""GPU parity of the on-the-fly weights that are laid out in memory (emb_kernels.hip): inputs beyond the range of the
exponentials, batches in slices, references whose cells crowd one tile, items computed by one workgroup, and
workspaces that only hold the kernels without weights in memory; against the float64 oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads
from gpu_util import announce, assert_dist_close, library_option
from test_gpu_fused import assert_grad_close, fused_inputs, run_fused_grads, run_fused_loss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", ["f", "e", "both", "infinite"])
def test_values_beyond_the_range_of_the_exponentials(case):
    """tanh(f + e) from e^2f e^2e: f or e alone far outside (saturated whatever the other is), both outside with sums
    of a few units, and infinities."""
    announce("wide inputs", case)
    s = workloads.shared_emb(B=3, T=9, V=5, order=2, H=128, seed=5, len_lo=6, len_hi=9)
    rng = np.random.default_rng(5)
    big = rng.choice([-1.0, 1.0], size=128) * rng.uniform(31.0, 90.0, size=128)
    f, e = (oracle_float(s[k]).copy() for k in "fe")
    on = rng.random(128) < 0.3
    if case in ("f", "both"):
        f[:, :, on] = big[on]
    if case == "e":
        e[:, on] = big[on]
    if case == "both":
        e[:, on] = -workloads_round(big)[on] + rng.standard_normal((e.shape[0], int(on.sum())))
    if case == "infinite":
        f[:, ::2, on] = np.inf
        f[:, 1::2, on] = -np.inf
    s["f"], s["e"] = workloads.to_bf16_bits(f.astype(np.float32)), workloads.to_bf16_bits(e.astype(np.float32))
    run_fused_grads(s)


def oracle_float(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32)


def workloads_round(x):
    return oracle_float(workloads.to_bf16_bits(x.astype(np.float32)))


@pytest.mark.parametrize("fill", [50.0, float("inf")])
def test_frames_past_the_end_have_no_part_in_the_results(fill):
    """Large values of e, and large ones of f only behind the ends of the items: the same bits as with zeros there."""
    announce("frames past the end", fill)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    B, T, V, H = 3, 40, 20, 128
    C = 1 + V + V * V
    f = torch.randn((B, T, H), generator=g, device="cuda")
    e = 0.5 * torch.randn((C, H), generator=g, device="cuda")
    e[:, ::8] = 35.0
    W = (torch.randn((H, V + 1), generator=g, device="cuda") / H ** 0.5).bfloat16()
    lengths = torch.tensor([T, 25, 0], dtype=torch.int32, device="cuda")
    got = []
    for x in (0.0, fill):
        f[1, 25:], f[2] = x, x
        dist, grads = lb.last_arc_posteriors(lb.SharedEmb(f.bfloat16(), e.bfloat16(), W), lengths, order=2)
        got.append((dist, *grads))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_hidden_units_of_sums_that_cancel():
    """tanh(f + e) of large f and e whose sum is 0.  e^2f and e^2e are rounded once each, so that their product is within
    2^-23 of 1; 1 more is 2, or 2 - 2^-23, in float32, and the tanh 0 or -2^-24.  Weights are such tanh times 64, 128 times,
    in every label but the empty one."""
    announce("sums that cancel")
    B, T, V, H = 16, 8, 3, 128
    C = 1 + V + V * V
    c = torch.linspace(2.5, 29.5, B, device="cuda").bfloat16()
    worst = 0.0
    for b in range(B):                                  # (e is shared by the items of a call)
        f = c[b].expand(1, T, H).contiguous()
        e = (-c[b]).expand(C, H).contiguous()
        W = torch.full((H, V + 1), 64.0, device="cuda").bfloat16()
        W[:, 0] = 0.0
        dist, _ = lb.last_arc_posteriors(lb.SharedEmb(f, e, W), torch.tensor([T], dtype=torch.int32, device="cuda"), order=2)
        worst = max(worst, abs(float(dist) / T - float(np.log(V + 1.0))))
    print("worst", worst, flush=True)
    # d log(1 + V e^w) = V / (V + 1) w for w = 64 H h
    assert worst <= V / (V + 1.0) * 64 * H * 2.0 ** -24, worst


def test_batch_in_slices_returns_what_its_items_return_alone():
    """Three items of which two fit the weights kept at a time: distances and df bit for bit those of calls with one
    item each, de and dW their sum."""
    B, T, V, H = 3, 3500, 64, 128
    announce("slices", B, T, V, H)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    C = 1 + V + V * V
    f = torch.randn((B, T, H), generator=g, device="cuda").bfloat16()
    e = (0.5 * torch.randn((C, H), generator=g, device="cuda")).bfloat16()
    W = (torch.randn((H, V + 1), generator=g, device="cuda") / H ** 0.5).bfloat16()
    lengths = torch.tensor([T, T - 77, T - 1200], dtype=torch.int32, device="cuda")
    d0 = lb.last_shortest_distance(lb.SharedEmb(f, e, W), lengths, order=2)
    dist, (df, de, dW) = lb.last_arc_posteriors(lb.SharedEmb(f, e, W), lengths, order=2)
    assert torch.equal(d0, dist)
    de1, dW1 = torch.zeros_like(de), torch.zeros_like(dW)
    for b in range(B):
        d1, (df1, x, y) = lb.last_arc_posteriors(lb.SharedEmb(f[b:b + 1].contiguous(), e, W), lengths[b:b + 1], order=2)
        assert torch.equal(d1, dist[b:b + 1])
        # (stretches of frames differ with the batch, sums over the states of a frame do not)
        assert torch.equal(df1[0], df[b])
        de1 += x
        dW1 += y
    assert_grad_close("de", de.cpu().numpy(), de1.cpu().numpy())
    assert_grad_close("dW", dW.cpu().numpy(), dW1.cpu().numpy())


@pytest.mark.parametrize("H,V,U", [(128, 3, 200), (512, 33, 40), (256, 32, 0)])
def test_loss_with_many_cells_in_one_tile(H, V, U):
    """References of one label over and over: all cells of the intersected lattice in one tile of states, more of them
    than a workgroup has threads (H = 128); no label at all; accumulated with a scale."""
    B, T = 2, max(30, U + 40)
    announce("cells of one tile", H, V, U)
    s = workloads.shared_emb(B=B, T=T, V=V, order=2, H=H, seed=9, len_lo=T - 5, len_hi=T)
    s["refs"] = np.full((B, max(U, 1)), 2, dtype=np.int32)
    s["ref_lengths"] = np.asarray([U, U // 2], dtype=np.int32)
    se = fused_inputs(s)
    st = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    grads = tuple(torch.full(t.shape, 3.0, dtype=torch.float32, device="cuda") for t in se)
    D, N, _ = lb.last_globally_normalized_loss(se, torch.from_numpy(s["lengths"]).cuda(), torch.from_numpy(s["refs"]).cuda(),
                                               torch.from_numpy(s["ref_lengths"]).cuda(), order=2, dw=grads, scale=0.5,
                                               accumulate=True, item_status=st)
    torch.cuda.synchronize()
    den = oracle.fused_forward_backward(s["f"], s["e"], s["W"], s["lengths"], 2, round_h=True, grads=True)
    num = oracle.fused_numerator(s["f"], s["e"], s["W"], s["lengths"], s["refs"], s["ref_lengths"], 2)
    assert st.cpu().tolist() == [0] * B
    assert_dist_close(D.cpu().numpy(), den["D"])
    assert_dist_close(N.cpu().numpy(), num["N"], "numerator")
    for name, got in zip(("df", "de", "dW"), grads):
        a, b = den[name].astype(np.float64), num[name].astype(np.float64)
        tol = 1e-4 * max(1.0, np.max(np.abs(a)) + np.max(np.abs(b)))      # a difference of two such terms
        assert np.max(np.abs(got.cpu().numpy() - (3.0 + 0.5 * (a - b)))) <= tol, name


@pytest.mark.parametrize("B,T,V,H,U", [(2, 24, 40, 128, 9), (4, 12, 4, 512, 6), (2, 60, 12, 128, 20)])
def test_loss_gradient_is_that_of_marginals_in_float32(B, T, V, H, U):
    """Marginals of the intersected lattice, near 1 on a few arcs, keep 24 bits on their way through the weight function.
    Bound: with float32 marginals 1.3e-7 to 3.9e-7 of the gradient's norm is left (root mean square over six inputs:
    exponentials of sums of a few dozen); a rounding of every marginal to 16 bits, 2^-18 of it at most and 0.6 of that
    on average, alone leaves 4e-7 (de) to 1.9e-6 (df)."""
    announce("precision of the loss gradient", B, T, V, H, U)
    sq = {"df": 0.0, "de": 0.0, "dW": 0.0}
    for seed in range(6):
        s = workloads.shared_emb(B=B, T=T, V=V, order=2, H=H, seed=seed, len_lo=T - 2, len_hi=T)
        s["refs"], s["ref_lengths"] = workloads.references(np.random.default_rng(seed), B, V, U, U - 2, U)
        lengths, refs, ulen = (torch.from_numpy(s[k]).cuda() for k in ("lengths", "refs", "ref_lengths"))
        _, _, grads = lb.last_globally_normalized_loss(fused_inputs(s), lengths, refs, ulen, order=2)
        den = oracle.fused_forward_backward(s["f"], s["e"], s["W"], s["lengths"], 2, round_h=True, grads=True)
        num = oracle.fused_numerator(s["f"], s["e"], s["W"], s["lengths"], s["refs"], s["ref_lengths"], 2)
        for name, got in zip(("df", "de", "dW"), grads):
            want = den[name].astype(np.float64) - num[name]
            sq[name] += (np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)) ** 2 / 6
    print({k: "%.2e" % x ** 0.5 for k, x in sq.items()}, flush=True)
    for name, most in (("df", 6e-7), ("de", 3.5e-7), ("dW", 5e-7)):
        assert sq[name] ** 0.5 <= most, (name, sq[name] ** 0.5)


def test_gradients_at_addresses_of_single_floats():
    """Only f, e and W have to lie on 16 bytes: gradients one float further on hold the same bits, and nothing beside them."""
    announce("gradients on 4 bytes")
    s = workloads.shared_emb(B=2, T=9, V=7, order=2, H=128, seed=12, len_lo=5, len_hi=9)
    se, lengths = fused_inputs(s), torch.from_numpy(s["lengths"]).cuda()
    for accumulate in (False, True):
        want = [torch.full(t.shape, 2.0, dtype=torch.float32, device="cuda") for t in se]
        flat = [torch.full((t.numel() + 2,), 2.0, dtype=torch.float32, device="cuda") for t in se]
        got = [x[1:-1].view(t.shape) for x, t in zip(flat, se)]
        assert all(x.data_ptr() % 16 == 4 for x in got)
        for grads in (want, got):
            lb.last_arc_posteriors(se, lengths, order=2, dw=tuple(grads), accumulate=accumulate)
        for x, y, z in zip(want, got, flat):
            assert torch.equal(x, y) and float(z[0]) == 2.0 and float(z[-1]) == 2.0


def test_items_whose_waits_ran_out_have_their_gradient():
    announce("spin limit 1, weights in memory")
    with library_option(lb.OPT_SPIN_LIMIT, 1):
        run_fused_grads(workloads.shared_emb(B=4, T=13, V=24, order=2, H=128, seed=78, len_lo=5, len_hi=13))


@pytest.mark.parametrize("V,lens", [(3, [1, 0, 2]), (31, [40, 0, 33]), (47, [7, 7, 1]), (64, [9, 2, 5])])
def test_lengths_labels_and_smaller_workspaces(V, lens):
    """Lengths of nothing and of one frame, tiles of labels with remainders; the entry point with the static workspace
    and the smallest workspace that the call takes, which holds no weights."""
    announce("lengths and workspaces", V, lens)
    s = workloads.shared_emb(B=3, T=max(lens), V=V, order=2, H=256, seed=V)
    s["lengths"] = np.asarray(lens, dtype=np.int32)
    o, _ = run_fused_grads(s)
    se, lengths = fused_inputs(s), torch.from_numpy(s["lengths"]).cuda()
    dist = torch.empty(3, dtype=torch.float32, device="cuda")
    lb.last_shortest_distance_static(se, lengths, dist, order=2)
    torch.cuda.synchronize()
    assert_dist_close(dist.cpu().numpy(), o["D"])
    wt, cx, _, _ = lb._weights_and_context(se, 2)
    with library_option(lb.OPT_FUSED_KEEP_MARGINALS, 0):
        small = lb.last_workspace_bytes(wt, cx, lb.OP_SHORTEST_DISTANCE)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    dist2 = torch.empty_like(dist)
    for nbytes, code in ((small, 0), (small - 1, 5)):
        assert lb.load_library().last_shortest_distance(
            ctypes.byref(wt), lb._ptr(lengths), ctypes.byref(cx), lb.LAST_LOG, lb._ptr(dist2), None, lb._ptr(ws), nbytes,
            lb._stream()) == code
    torch.cuda.synchronize()
    assert_dist_close(dist2.cpu().numpy(), o["D"])


def test_calls_on_a_card_without_room_for_the_weights():
    """The binding asks for 0.5 to 2.3 GiB of scratch where the allocator may give 300 MiB: the calls go through with the
    kernels that hold no weights, and nothing of the smaller buffers is kept."""
    announce("no room for the weights")
    s = workloads.shared_emb(B=2, T=240, V=64, order=2, H=128, seed=4, len_lo=200, len_hi=240)
    s["refs"], s["ref_lengths"] = workloads.references(np.random.default_rng(4), 2, 64, 30, 10, 30)
    se = fused_inputs(s)
    lengths, refs, ulen = (torch.from_numpy(s[k]).cuda() for k in ("lengths", "refs", "ref_lengths"))

    def calls():
        d0 = lb.last_shortest_distance(se, lengths, order=2)
        d1, g1 = lb.last_arc_posteriors(se, lengths, order=2)
        lb.check_item_status()
        d2, n2, g2 = lb.last_globally_normalized_loss(se, lengths, refs, ulen, order=2)
        lb.check_item_status()
        return [t.cpu().numpy() for t in (d0, d1, *g1, d2, n2, *g2)]
    want = calls()
    lb.release_workspaces()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (300 << 20)) / total)
    try:
        got = calls()
        assert not lb._workspaces
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    for a, b in zip(got, want):
        assert_grad_close("one result", a, b)


@pytest.mark.parametrize("force_solo", [0, 1])
@pytest.mark.parametrize("V,lens,U", [(2, [6, 3], 3), (3, [9, 0], 4), (33, [7, 6], 5)])
def test_gradients_in_smaller_workspaces(V, lens, U, force_solo):
    """Posteriors and loss take a workspace that only holds the kernels without weights, and without marginals kept between
    two of them: the size asked for with LAST_OPT_FUSED_KEEP_MARGINALS = 0, used with 1; a byte less is refused."""
    announce("gradients, smaller workspace", V, lens, U, force_solo)
    B, H = 2, 256
    s = workloads.shared_emb(B=B, T=max(lens), V=V, order=2, H=H, seed=V)
    s["lengths"] = np.asarray(lens, dtype=np.int32)
    s["refs"], s["ref_lengths"] = workloads.references(np.random.default_rng(V), B, V, U, 0, min(U, *lens))
    se = fused_inputs(s)
    lengths, refs, ulen = (torch.from_numpy(s[k]).cuda() for k in ("lengths", "refs", "ref_lengths"))
    den = oracle.fused_forward_backward(s["f"], s["e"], s["W"], s["lengths"], 2, round_h=True, grads=True)
    num = oracle.fused_numerator(s["f"], s["e"], s["W"], s["lengths"], s["refs"], s["ref_lengths"], 2)
    wt, cx, _, _ = lb._weights_and_context(se, 2)
    lib = lb.load_library()
    with library_option(lb.OPT_FUSED_KEEP_MARGINALS, 0):
        least = lb.last_workspace_bytes(wt, cx, lb.OP_ARC_POSTERIORS)
    beside = lb.last_workspace_bytes(wt, cx, lb.OP_INTERSECT_REFERENCE, U)
    assert lib.last_least_workspace_bytes(ctypes.byref(wt), ctypes.byref(cx), lb.OP_ARC_POSTERIORS, 0) == least
    assert lib.last_least_workspace_bytes(ctypes.byref(wt), ctypes.byref(cx), lb.OP_LOSS, U) == least + beside
    ws = torch.empty(least + beside, dtype=torch.uint8, device="cuda")
    grads = [torch.empty(t.shape, dtype=torch.float32, device="cuda") for t in se]
    g = lb.LastGrads(None, *(t.data_ptr() for t in grads), 0, 1.0)
    dist, score = (torch.empty(B, dtype=torch.float32, device="cuda") for _ in range(2))
    args = ctypes.byref(wt), lb._ptr(lengths), ctypes.byref(cx)
    with library_option(lb.OPT_FORCE_SOLO, force_solo):
        for nbytes, code in ((least - 1, 5), (least, 0)):
            assert lib.last_arc_posteriors(*args, lb._ptr(dist), ctypes.byref(g), None, lb._ptr(ws), nbytes, lb._stream()) == code
        torch.cuda.synchronize()
        assert_dist_close(dist.cpu().numpy(), den["D"])
        for name, got in zip(("df", "de", "dW"), grads):
            assert_grad_close(name, got.cpu().numpy(), den[name])
        for nbytes, code in ((least + beside - 1, 5), (least + beside, 0)):
            assert lib.last_globally_normalized_loss(*args, lb._ptr(refs), lb._ptr(ulen), U, lb._ptr(dist), lb._ptr(score),
                                                     ctypes.byref(g), None, lb._ptr(ws), nbytes, lb._stream()) == code
        torch.cuda.synchronize()
    assert_dist_close(dist.cpu().numpy(), den["D"])
    assert_dist_close(score.cpu().numpy(), num["N"], "numerator")
    for name, got in zip(("df", "de", "dW"), grads):
        a, b = den[name].astype(np.float64), num[name].astype(np.float64)
        tol = 1e-4 * max(1.0, np.max(np.abs(a)) + np.max(np.abs(b)))      # a difference of two such terms
        assert np.max(np.abs(got.cpu().numpy() - (a - b))) <= tol, name
