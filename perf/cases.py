"""The workloads by which the speed of this library is judged: what a training or decoding program
asks of it, through the calls of ``paper_2304_13134_amd.binding``.

A case is a dict of plain values:

    op       "loss"        last_globally_normalized_loss (a training step's lattice work)
             "posteriors"  last_arc_posteriors (forward-backward alone)
             "local"       last_local_log_likelihood with its gradient (the locally normalised loss)
             "distance"    last_shortest_distance, log semiring (scoring, a validation pass)
             "path"        last_shortest_path (decoding)
    context  "bigram", "trigram" (closed form), "ngram3" (contexts of up to three labels, as a
             next-state table), "automaton" (any deterministic automaton with `C` states, as a table)
    H        0: dense weights [B,T,C,V+1]; otherwise the on-the-fly weights tanh(f+e) @ W of that width
    B, T, V  items, frames, labels; lengths are drawn from [len_lo, T]
    U_lo, U_hi   range of the reference lengths (loss, local)
    sigma    standard deviation of dense weights
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2304_13134_amd import binding as lb
from paper_2304_13134_amd import workloads


def _case(name, op, context, B, T, V, len_lo=None, H=0, U=(0, 0), sigma=1.0, C=0):
    return {"name": name, "op": op, "context": context, "B": B, "T": T, "V": V,
            "len_lo": T if len_lo is None else len_lo, "H": H, "U_lo": U[0], "U_hi": U[1],
            "sigma": sigma, "C": C or _closed_states(context, V)}


def _closed_states(context, V):
    return sum(V ** k for k in range({"bigram": 1, "trigram": 2, "ngram3": 3}[context] + 1))


def listed():
    return [
        # the smallest lattice of the tests and examples: one short item, where launches are all there is
        _case("posteriors_bigram_tiny", "posteriors", "bigram", B=1, T=8, V=3),
        # a training step of a small character model: 32 labels, a small batch of utterances of unequal length
        _case("loss_bigram_characters", "loss", "bigram", B=8, T=200, V=32, len_lo=150, U=(10, 60)),
        # a training step with 256 subword labels at full batch, the benchmark's dense lattice
        _case("loss_bigram_subwords", "loss", "bigram", B=16, T=500, V=256, U=(50, 150), sigma=2.0),
        # forward-backward with a label set that no tile divides and ragged lengths, more items than clusters
        _case("posteriors_bigram_ragged", "posteriors", "bigram", B=20, T=333, V=130, len_lo=100, sigma=1.5),
        # batch decoding with 256 subword labels
        _case("path_bigram_subwords", "path", "bigram", B=16, T=500, V=256, sigma=2.0),
        # interactive decoding: one short utterance, character labels
        _case("path_bigram_one_utterance", "path", "bigram", B=1, T=150, V=47),
        # a training step of the two-label context on weights that the model has laid out in memory
        _case("loss_trigram_dense", "loss", "trigram", B=8, T=300, V=32, len_lo=200, U=(20, 100)),
        # batch decoding with the two-label context
        _case("path_trigram_dense", "path", "trigram", B=6, T=250, V=28, len_lo=120, sigma=1.5),
        # a training step with contexts of three labels (585 states), which only a next-state table expresses
        _case("loss_table_3gram", "loss", "ngram3", B=8, T=200, V=8, len_lo=120, U=(20, 80)),
        # the training step of the paper's benchmark: 32 labels, two-label context, on-the-fly weights
        _case("loss_shared_emb_characters", "loss", "trigram", B=16, T=1024, V=32, H=512, U=(256, 256)),
        # scoring with 64 labels on on-the-fly weights (a validation pass)
        _case("distance_shared_emb_64", "distance", "trigram", B=4, T=1000, V=64, H=512),
        # the locally normalised loss with gradient at 256 labels
        _case("local_bigram_subwords", "local", "bigram", B=16, T=500, V=256, U=(50, 150), sigma=2.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges: any operation on any context, sizes spread over their logarithm
    and scaled down until the case is no larger than the largest listed one of its kind."""
    context = rng.choice(["bigram", "bigram", "trigram", "table", "shared"])
    H, C = 0, 0
    if context == "bigram":
        V, T, B, arcs = _log_int(rng, 3, 260), _log_int(rng, 8, 600), _log_int(rng, 1, 32), 5.2e8
    elif context == "trigram":
        V, T, B, arcs = _log_int(rng, 4, 36), _log_int(rng, 8, 400), _log_int(rng, 1, 24), 8.0e7
    elif context == "table":
        context = rng.choice(["ngram3", "automaton"])
        T, B, arcs = _log_int(rng, 8, 300), _log_int(rng, 1, 24), 9.0e6
        V = _log_int(rng, 3, 9) if context == "ngram3" else _log_int(rng, 4, 60)
        C = _log_int(rng, 20, 1200) if context == "automaton" else 0
    else:
        context, H = "trigram", 128 * rng.randint(1, 4)
        V, T, B, arcs = _log_int(rng, 8, 64), _log_int(rng, 16, 1024), _log_int(rng, 1, 16), 3.0e8
    states = C or _closed_states(context, V)
    while B * T * states * (V + 1) > arcs:
        if B > 1 and (B > T // 16 or T <= 8):
            B -= max(1, B // 8)
        else:
            T -= max(1, T // 8)
    if context in ("ngram3", "automaton"):
        ops = ["loss", "posteriors", "path", "distance"]
    elif H:
        ops = ["loss", "posteriors", "distance"]
    else:
        ops = ["loss", "posteriors", "path", "distance", "local"]
    len_lo = rng.choice([T, max(1, T // 2), max(1, 3 * T // 4)])
    U_hi = rng.randint(max(1, len_lo // 8), max(1, len_lo // 2))
    return {"op": rng.choice(ops), "context": context, "B": B, "T": T, "V": V, "len_lo": len_lo, "H": H,
            "U_lo": max(1, U_hi // 3), "U_hi": U_hi, "sigma": round(rng.uniform(0.5, 2.0), 2), "C": states}


# ---- inputs ---------------------------------------------------------------------------------

def _ngram3_table(V):
    """table [C, V]: states are the label strings of length 0 to 3, ordered by length, then by label."""
    first = [0, 1, 1 + V, 1 + V + V * V]
    C = first[3] + V ** 3
    table = np.empty((C, V), np.int32)
    y = np.arange(V)
    for n in range(3):                                   # a shorter string grows by the label
        k = np.arange(V ** n)
        table[first[n]:first[n] + V ** n] = first[n + 1] + k[:, None] * V + y
    k = np.arange(V ** 3)                                # a string of three drops its oldest label
    table[first[3]:] = first[3] + (k % (V * V))[:, None] * V + y
    return table


def _table(case, seed):
    if case["context"] == "ngram3":
        return _ngram3_table(case["V"])
    return workloads.random_table(case["C"], case["V"], seed)


def _order(case, table):
    return {"bigram": 1, "trigram": 2}.get(case["context"], table)


def prepare(case, seed):
    B, T, V, C, H = case["B"], case["T"], case["V"], case["C"], case["H"]
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    st = {"op": case["op"], "case": case,
          "lengths": torch.from_numpy(rng.integers(case["len_lo"], T + 1, size=B).astype(np.int32)).cuda()}
    if case["op"] in ("loss", "local"):
        ulen = rng.integers(case["U_lo"], case["U_hi"] + 1, size=B).astype(np.int32)
        refs = rng.integers(1, V + 1, size=(B, case["U_hi"])).astype(np.int32)
        st["refs"], st["ref_lengths"] = torch.from_numpy(refs).cuda(), torch.from_numpy(ulen).cuda()
    table = None
    if case["context"] in ("ngram3", "automaton"):
        table = torch.from_numpy(_table(case, seed)).cuda()
    st["order"] = _order(case, table)
    if H:
        f = torch.randn((B, T, H), generator=g, device="cuda")
        e = torch.randn((C, H), generator=g, device="cuda") * 0.5
        W = torch.randn((H, V + 1), generator=g, device="cuda") / math.sqrt(H)
        st["w"] = lb.SharedEmb(f.bfloat16(), e.bfloat16(), W.bfloat16())
    else:
        st["w"] = torch.randn((B, T, C, V + 1), generator=g, device="cuda")
        st["w"] *= case["sigma"]
    return st


def run(state):
    op, w, lengths, order = state["op"], state["w"], state["lengths"], state["order"]
    if op == "loss":
        dist, num, grad = lb.last_globally_normalized_loss(w, lengths, state["refs"], state["ref_lengths"], order=order)
        return [dist, num, *(grad if isinstance(grad, tuple) else (grad,))]
    if op == "posteriors":
        dist, grad = lb.last_arc_posteriors(w, lengths, order=order)
        return [dist, *(grad if isinstance(grad, tuple) else (grad,))]
    if op == "local":
        grad = torch.empty_like(w)
        loglik = lb.last_local_log_likelihood(w, lengths, state["refs"], state["ref_lengths"], order=order, dw=grad)
        return [loglik, grad]
    if op == "distance":
        return [lb.last_shortest_distance(w, lengths, order=order)]
    return list(lb.last_shortest_path(w, lengths, order=order))


# ---- what a pass cannot do without --------------------------------------------------------------

def work(case):
    B, T, V, C, H, op = case["B"], case["T"], case["V"], case["C"], case["H"], case["op"]
    frames = B * 0.5 * (case["len_lo"] + T)              # frames that exist, on average
    arcs = frames * C * (V + 1)
    U = 0.5 * (case["U_lo"] + case["U_hi"])
    cells = frames * (U + 1)                             # states of the intersected lattice
    table = C * V * 4 if case["context"] in ("ngram3", "automaton") else 0
    if H:
        inputs = 2 * (B * T * H + C * H + H * (V + 1))
        if op == "distance":
            return {"bytes": inputs, "flops": arcs * 2 * H + frames * C * H}
        grads = 4 * (B * T * H + C * H + H * (V + 1))
        num = cells * 12 * H if op == "loss" else 0      # two arcs per state, three contractions each
        return {"bytes": inputs + grads, "flops": arcs * 6 * H + frames * C * H + num}
    if op == "local":                                    # rows that the reference visits; the gradient is written whole
        rows = frames * min(U + 1, C)
        return {"bytes": rows * (V + 1) * 4 + B * T * C * (V + 1) * 4, "flops": rows * (V + 1) * 4}
    if op == "distance":
        return {"bytes": arcs * 4 + table, "flops": arcs * 3}
    if op == "path":
        return {"bytes": arcs * 4 + table + B * (2 * T + 1) * 4, "flops": arcs * 2}
    return {"bytes": arcs * 4 + table + B * T * C * (V + 1) * 4,
            "flops": arcs * 8 + (cells * 12 if op == "loss" else 0)}


def tolerance(case):
    if case["op"] == "path":
        return "exact"          # one float32 add per arc in path order, ties to the lowest arc: bit-reproducible
    # Gradients are float32 exponentials of sums that reach several thousand.  Against 64 bits the relative
    # 2-norm of the error is 0.2e-6 to 1e-6, over the ranges of draw() up to 3.5e-6; distances are at 3e-8.
    # With on-the-fly weights a hidden unit next to a rounding boundary may round the other way: up to 3e-6.
    return {"rel": 1.5e-5}


# ---- the same in 64 bits, frame by frame ----------------------------------------------------------

def _next_states(case, seed):
    """next [C, V+1]: destination of every arc; label 0 keeps the state."""
    V, C = case["V"], case["C"]
    q, y = np.arange(C)[:, None], np.arange(1, V + 1)[None, :]
    if case["context"] == "bigram":
        nx = np.broadcast_to(y, (C, V))
    elif case["context"] == "trigram":
        last = np.where(q <= V, q, (q - 1 - V) % V + 1)
        nx = np.where(q == 0, y, 1 + V + (last - 1) * V + (y - 1))
    else:
        nx = _table(case, seed)
    return torch.from_numpy(np.concatenate([q, nx], axis=1).astype(np.int64)).cuda()


def _arrive(case, nx, s, best=False):
    """(+)-sum (log-add-exp, or the maximum) of the arc scores s [B, C, V+1] per destination state."""
    B, C, V = s.shape[0], case["C"], case["V"]
    reduce = (lambda x: x.amax(dim=1)) if best else (lambda x: torch.logsumexp(x, dim=1))
    both = torch.maximum if best else torch.logaddexp
    out = s[:, :, 0].clone()
    if case["context"] == "bigram":
        out[:, 1:] = both(out[:, 1:], reduce(s[:, :, 1:]))
    elif case["context"] == "trigram":
        out[:, 1:V + 1] = both(out[:, 1:V + 1], s[:, 0, 1:])
        by_last = torch.cat([s[:, 1:V + 1, 1:].reshape(B, 1, V, V), s[:, V + 1:, 1:].reshape(B, V, V, V)], dim=1)
        out[:, V + 1:] = both(out[:, V + 1:], reduce(by_last).reshape(B, V * V))
    else:
        to, flat = nx.reshape(1, -1).expand(B, -1), s.reshape(B, -1)
        top = torch.full((B, C), -math.inf, dtype=s.dtype, device=s.device).scatter_reduce(1, to, flat, "amax")
        if best:
            return top
        safe = torch.where(torch.isinf(top), torch.zeros_like(top), top)
        total = torch.zeros_like(top).scatter_add(1, to, torch.exp(flat - safe.gather(1, to)))
        out = safe + torch.log(total)
    return out


def _weights(st, t):
    """(weights of frame t in 64 bits [B, C, V+1], hidden vectors [B*C, H] or None)."""
    if not isinstance(st["w"], lb.SharedEmb):
        return st["w"][:, t].double(), None
    f, e, W = st["w"]
    x = f[:, t].float()[:, None, :] + e.float()[None, :, :]
    h = torch.tanh(x.double()).bfloat16().double().reshape(-1, f.shape[2])      # the hidden vector is bfloat16
    return (h @ W.double()).reshape(f.shape[0], e.shape[0], W.shape[1]), h


def exact(case, seed):
    st = prepare(case, seed)
    op, B, T, C = case["op"], case["B"], case["T"], case["C"]
    nx, lengths = _next_states(case, seed), st["lengths"].long()
    f64 = dict(dtype=torch.float64, device="cuda")
    dist = num = None
    start = torch.full((B, C), -math.inf, **f64)
    start[:, 0] = 0.0
    referenced = op in ("loss", "local")
    if referenced:
        refs, ulen = st["refs"].long(), st["ref_lengths"].long()
        U = refs.shape[1]
        cx = torch.zeros((B, U + 1), dtype=torch.int64, device="cuda")         # context after u labels
        for u in range(U):
            cx[:, u + 1] = nx[cx[:, u], refs[:, u]]
        item = torch.arange(B, device="cuda")[:, None]
        label = torch.cat([refs, refs[:, :1]], dim=1)                          # (the last one is never taken)
        wblank, wlabel, lz = (torch.empty((T, B, U + 1), **f64) for _ in range(3))
    # forward
    alpha = [start]
    for t in range(T):
        w, _ = _weights(st, t)
        if referenced:
            wblank[t], wlabel[t] = w[item, cx, 0], w[item, cx, label]
            if op == "local":
                lz[t] = torch.logsumexp(w, dim=2)[item, cx]
                wblank[t] -= lz[t]
                wlabel[t] -= lz[t]
        if op != "local":
            here = (t < lengths)[:, None]
            alpha.append(torch.where(here, _arrive(case, nx, alpha[-1][:, :, None] + w, best=op == "path"), alpha[-1]))
    if op == "path":
        return [None, None, alpha[-1].amax(dim=1)]
    if op != "local":
        dist = torch.logsumexp(alpha[-1], dim=1)
    if op == "distance":
        return [dist]
    if referenced:
        live = torch.arange(U + 1, device="cuda")[None, :] <= ulen[:, None]
        can = torch.arange(U + 1, device="cuda")[None, :] < ulen[:, None]       # a label is left to read
        none = torch.full((B, 1), -math.inf, **f64)
        inf = torch.full((B, U + 1), -math.inf, **f64)
        a = [torch.where(torch.arange(U + 1, device="cuda")[None, :] == 0, 0.0, inf)]
        for t in range(T):
            stay = a[-1] + wblank[t]
            go = torch.where(can, a[-1] + wlabel[t], inf)
            new = torch.where(live, torch.logaddexp(stay, torch.cat([none, go[:, :-1]], dim=1)), inf)
            a.append(torch.where((t < lengths)[:, None], new, a[-1]))
        num = a[-1].gather(1, ulen[:, None])[:, 0]
        done = torch.where(torch.arange(U + 1, device="cuda")[None, :] == ulen[:, None], 0.0, inf)
        bk = done
    # backward
    beta = torch.zeros((B, C), **f64)
    shared = isinstance(st["w"], lb.SharedEmb)
    if shared:
        f, e, W = st["w"]
        W64 = W.double()
        df, de, dW = (torch.zeros(x.shape, **f64) for x in (f, e, W))
    else:
        grad = torch.zeros(st["w"].shape, **f64)
    for t in range(T - 1, -1, -1):
        here = (t < lengths)[:, None]
        w, h = _weights(st, t)
        gamma = torch.zeros_like(w)
        if op != "local":
            s = w + beta[:, nx]
            gamma = torch.where(here[:, :, None], torch.exp(alpha[t][:, :, None] + s - dist[:, None, None]), 0.0)
            beta = torch.where(here, torch.logsumexp(s, dim=2), beta)
        if referenced:
            stay = wblank[t] + bk
            go = torch.where(can, wlabel[t] + torch.cat([bk[:, 1:], none], dim=1), inf)
            gblank = torch.where(here, torch.exp(a[t] + stay - num[:, None]), 0.0)
            glabel = torch.where(here, torch.exp(a[t] + go - num[:, None]), 0.0)
            bk = torch.where(here, torch.logaddexp(stay, go), bk)
            sign = 1.0 if op == "local" else -1.0
            gamma.index_put_((item.expand_as(cx), cx, torch.zeros_like(cx)), sign * gblank, accumulate=True)
            gamma.index_put_((item.expand_as(cx), cx, label), sign * glabel, accumulate=True)
            if op == "local":
                occupied = torch.zeros((B, C), **f64)
                occupied.index_put_((item.expand_as(cx), cx), gblank + glabel, accumulate=True)
                gamma -= occupied[:, :, None] * torch.softmax(w, dim=2)
        if shared:
            flat = gamma.reshape(-1, gamma.shape[2])
            dpre = ((flat @ W64.t().contiguous()) * (1.0 - h * h)).reshape(B, C, -1)
            df[:, t] = dpre.sum(dim=1)
            de += dpre.sum(dim=0)
            dW += h.t() @ flat
        else:
            grad[:, t] = gamma
    grads = [df, de, dW] if shared else [grad]
    return [x for x in (dist, num) if x is not None] + grads
