// The recursions for a context dependency given as a next-state table, both
// directions at once (one workgroup per item and direction), for frames of up
// to 16384 arcs; larger ones take table_kernels.hpp / solo_kernels.hpp.
//
// The forward direction pushes arcs into their destinations with the same
// order-independent LDS atomics as table_forward_log (maximum, then fixed-point
// sum; tropical: one 64-bit maximum), so results do not depend on timing.  What
// bound that kernel (12 us a frame at 585 states, 9 labels) was the latency of
// its loads: weights and table entries were fetched where they were used, twice a
// frame.  Here a thread owns the same 16-byte pieces of every frame, keeps the
// source and destination of their arcs in registers for the whole item, and
// requests its weights two frames ahead; a frame is a chain of four barriers.
// The backward direction reduces rows: the pieces go through LDS, together with
// the table's entries as 16-bit numbers, and LPR lanes take a row.
// Measured (8 items, 120 to 200 frames, 585 states, 8 labels): both directions 2.4 us a
// frame, the loss with gradient 0.53 ms against 6.0 ms.
// Natural logs relative to a float64 offset per frame, rounded as in table_kernels.hpp; marginals are formed from the
// stored vectors by dense_marginals_kernel.
#pragma once
#include "common.hpp"
#include "table_kernels.hpp"
#include "trigram_kernels.hpp"

namespace last {

struct TabArgs {
    const float* w;
    const int* len;
    const int* bad;      // set by table_check_kernel; null for a closed-form context
    float* alpha;        // rows of C floats; tropical: unused
    float* beta;
    double* offa;
    double* offb;
    double* D2;
    float* dist;
    int* item_status;
    int* bp;             // tropical (may be null)
    int* final_state;
    int T, keep, lpr;    // keep: rows of every frame and the distance; lpr: lanes per row, backward
};

constexpr int kTabThreads = 1024;
constexpr int kTabMaxQ = 4;          // 16-byte pieces per thread: 16384 arcs

// LDS bytes of either direction
__host__ __device__ inline size_t tab_lds(int C, int V1, bool trop)
{
    const size_t n = (size_t)C * V1;
    const size_t fwd = (size_t)C * (trop ? 12 : 16) + 64 * sizeof(float);
    const size_t bwd = ((n + 7) & ~(size_t)3) * 4 + ((n + 3) & ~(size_t)3) * 2 + (size_t)C * 8 + 64 * sizeof(float);
    return trop || fwd > bwd ? fwd : bwd;
}

// log(sum 2^-40) of a fixed-point sum: exponent, mantissa in [0.7, 1.4) and what the mantissa was rounded by apart, so
// that the result is as good as the double-precision logarithm rounded to float32 (which took a fifth of a frame here)
__device__ __forceinline__ float tab_ln(tk_u64 sum)
{
    const double d = (double)sum * kTkUnfix;
    const float f = (float)d;
    int e = __builtin_amdgcn_frexp_expf(f);
    float m = __builtin_amdgcn_frexp_mantf(f);
    const bool low = m < 0.70710678f;
    m = low ? 2.f * m : m;
    e -= low;
    const float r = (float)(d - (double)f) * __builtin_amdgcn_rcpf(f);
    return fmaf((float)e, kLn2, fmaf(__builtin_amdgcn_logf(m), kLn2, r));
}

// largest value of the workgroup's 16 waves; ends with the barrier after which red is readable
__device__ __forceinline__ float tab_block_max(float v, float* red)
{
    v = wave_max_dpp(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    lds_only_barrier();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < kTabThreads / kWave; ++i) r = fmaxf(r, red[i]);
    return r;
}

template <int NQ, bool TROP>
__global__ __launch_bounds__(kTabThreads) void table_chain_kernel(TabArgs a, Ctx c)
{
    extern __shared__ __align__(16) tk_u64 tab_s[];
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool back = !TROP && blockIdx.y == 1;
    const int C = c.C, V1 = c.V1, n = C * V1;
    const int L = a.len[b];
    const bool badtab = a.bad && a.bad[0] != 0;
    if (L < 0 || L > a.T || badtab) {
        if ((TROP || a.keep) && !back && tid == 0) {
            a.dist[b] = __builtin_nanf("");
            if (!TROP) a.D2[b] = __builtin_nan("");
            if (TROP && a.final_state) a.final_state[b] = -1;
            if (a.item_status) a.item_status[b] = badtab ? kItemBadTable : kItemBadLength;
        }
        return;
    }
    const int low = a.keep ? 1 : L / 2;
    const int steps = TROP ? L : back ? max(L - low, 0) : a.keep ? L : L / 2;
    const float* wi = a.w + (size_t)b * a.T * n;
    // piece j of a thread: arcs pf[j] .. pf[j] + 3 of a frame (the last one ends with the frame; the arcs it shares with
    // the piece before it, and whole pieces past the end, do not count)
    int pf[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) pf[j] = min(4 * (tid + kTabThreads * j), n - 4);
    float4 raw[2][NQ];
    auto issue = [&](auto S, int k) __attribute__((always_inline)) {
        const int t = back ? max(L - 1 - k, 0) : min(k, max(L - 1, 0));
        const buf_t rs = make_buf(wi + (size_t)t * n, 4u * (unsigned)n);
#pragma unroll
        for (int j = 0; j < NQ; ++j) raw[decltype(S)::value][j] = tri_load4(rs, 4u * (unsigned)pf[j], 0);
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    if (steps > 0) {
        issue(I0(), 0);
        issue(I1(), 1);
    }

    if (!back) {
        tk_u64* sm = tab_s;                                  // fixed-point sums (tropical: keys)
        float* cur = (float*)(sm + C);
        int* mk = (int*)(cur + C);                           // log: keys of the maxima
        float* red = TROP ? (float*)(cur + C) : (float*)(mk + C);
        const int kneg = tk_skey(LAST_NEG_INF);
        const tk_u64 knone = (tk_u64)tk_ukey(LAST_NEG_INF) << 32;
        unsigned arc[NQ][4];                                 // destination | source << 16; all ones: no arc
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            int q = pf[j] / V1, y = pf[j] - q * V1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool counts = pf[j] + k >= 4 * (tid + kTabThreads * j);
                arc[j][k] = counts ? (unsigned)ctx_next(c, q, y) | ((unsigned)q << 16) : 0xffffffffu;
                const bool wrap = ++y == V1;
                q += wrap;
                y = wrap ? 0 : y;
            }
        }
        double A = 0.0;
        for (int d = tid; d < C; d += kTabThreads) {
            cur[d] = d == 0 ? 0.f : LAST_NEG_INF;
            if (TROP) sm[d] = knone;
            else { sm[d] = 0; mk[d] = kneg; }
        }
        __syncthreads();
        auto frame = [&](auto S, int t) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            float v[NQ][4];
#pragma unroll
            for (int j = 0; j < NQ; ++j) {
                const float wv[4] = {raw[Z][j].x, raw[Z][j].y, raw[Z][j].z, raw[Z][j].w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool on = arc[j][k] != 0xffffffffu;
                    const float x = on ? cur[arc[j][k] >> 16] : LAST_NEG_INF;
                    // (an arc out of an unreachable state does not count, whatever its weight)
                    v[j][k] = x == LAST_NEG_INF ? LAST_NEG_INF : __fadd_rn(x, wv[k]);
                }
            }
#pragma unroll
            for (int j = 0; j < NQ; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (v[j][k] != LAST_NEG_INF) {
                        if (TROP) {
                            const unsigned flat = (unsigned)(pf[j] + k);
                            atomicMax(&sm[arc[j][k] & 0xffffu], ((tk_u64)tk_ukey(v[j][k]) << 32) | (0xFFFFFFFFu - flat));
                        } else {
                            atomicMax(&mk[arc[j][k] & 0xffffu], tk_skey(v[j][k]));
                        }
                    }
            issue(S, t + 2);
            lds_only_barrier();
            if (TROP) {
                for (int d = tid; d < C; d += kTabThreads) {
                    const tk_u64 k = sm[d];
                    const unsigned lo = (unsigned)k;
                    cur[d] = lo == 0u ? LAST_NEG_INF : tk_uval((unsigned)(k >> 32));
                    sm[d] = knone;
                    if (a.bp) a.bp[((size_t)b * a.T + t) * C + d] = lo == 0u ? -1 : (int)(0xFFFFFFFFu - lo);
                }
                lds_only_barrier();
                return;
            }
#pragma unroll
            for (int j = 0; j < NQ; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (v[j][k] != LAST_NEG_INF) {
                        const int d = arc[j][k] & 0xffffu;
                        atomicAdd(&sm[d], (tk_u64)(tri_exp(v[j][k] - tk_sval(mk[d])) * kTkFix));
                    }
            lds_only_barrier();
            float mx = LAST_NEG_INF;
            for (int d = tid; d < C; d += kTabThreads) {
                const float m = tk_sval(mk[d]);
                const float x = m == LAST_NEG_INF ? m : m + tab_ln(sm[d]);
                cur[d] = x;
                mk[d] = kneg;
                sm[d] = 0;
                mx = fmaxf(mx, x);
            }
            mx = tab_block_max(mx, red);
            if (mx == LAST_NEG_INF) mx = 0.f;                // no state reachable: keep -inf everywhere
            A += (double)mx;
            for (int d = tid; d < C; d += kTabThreads) {
                const float x = cur[d] - mx;
                cur[d] = x;
                if (a.keep) a.alpha[((size_t)b * (a.T + 1) + t + 1) * C + d] = x;
            }
            if (a.keep && tid == 0) a.offa[(size_t)b * (a.T + 1) + t + 1] = A;
            lds_only_barrier();
        };
        if (!TROP && a.keep) {
            for (int d = tid; d < C; d += kTabThreads) a.alpha[(size_t)b * (a.T + 1) * C + d] = cur[d];
            if (tid == 0) a.offa[(size_t)b * (a.T + 1)] = 0.0;
        }
        for (int t = 0; t < steps; t += 2) {
            frame(I0(), t);
            if (t + 1 < steps) frame(I1(), t + 1);
        }
        if (TROP) {
            float best = LAST_NEG_INF;
            int bidx = 0x7fffffff;
            for (int d = tid; d < C; d += kTabThreads)
                if (cur[d] > best || (cur[d] == best && d < bidx)) { best = cur[d]; bidx = d; }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float ov = __shfl_xor(best, o, kWave);
                const int oi = __shfl_xor(bidx, o, kWave);
                if (ov > best || (ov == best && oi < bidx)) { best = ov; bidx = oi; }
            }
            int* redi = (int*)(red + 32);
            if ((tid & 63) == 0) { red[tid >> 6] = best; redi[tid >> 6] = bidx; }
            __syncthreads();
            if (tid == 0) {
                for (int k = 1; k < kTabThreads / kWave; ++k)
                    if (red[k] > best || (red[k] == best && redi[k] < bidx)) { best = red[k]; bidx = redi[k]; }
                a.dist[b] = best;
                if (a.final_state) a.final_state[b] = bidx;
                if (a.item_status) a.item_status[b] = kItemOk;
            }
        } else if (!a.keep) {
            for (int d = tid; d < C; d += kTabThreads) a.alpha[(size_t)b * C + d] = cur[d];
            if (tid == 0) a.offa[b] = A;
        } else {
            // all states of the last frame are final with weight 0; cur is relative to its largest entry
            float mx = LAST_NEG_INF;
            for (int d = tid; d < C; d += kTabThreads) mx = fmaxf(mx, cur[d]);
            mx = tab_block_max(mx, red);
            const float mm = mx == LAST_NEG_INF ? 0.f : mx;
            double z = 0.0;
            for (int d = tid; d < C; d += kTabThreads) z += (double)tri_exp(cur[d] - mm);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
            __syncthreads();
            double* redd = (double*)tab_s;                   // (the sums are done with)
            if ((tid & 63) == 0) redd[tid >> 6] = z;
            __syncthreads();
            if (tid == 0) {
                z = 0.0;
                for (int k = 0; k < kTabThreads / kWave; ++k) z += redd[k];
                const double d2 = mx == LAST_NEG_INF ? (double)LAST_NEG_INF : A + (double)mm + log(z);
                a.D2[b] = d2;
                a.dist[b] = (float)d2;
                if (a.item_status) a.item_status[b] = kItemOk;
            }
        }
        return;
    }

    // backward: rows
    float* tile = (float*)tab_s;                             // [n] weights of a frame
    float* be = tile + ((n + 7) & ~3);                       // [C] the vector of the frame after it
    float* bc = be + C;                                      // [C] the new one before its offset is taken out
    float* red = bc + C;
    unsigned short* nxs = (unsigned short*)(red + 64);       // [n] destinations
    auto spread = [&](auto S) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            if (4 * (tid + kTabThreads * j) >= n) continue;
            float* d = tile + pf[j];
            const float4 x = raw[decltype(S)::value][j];
            if (pf[j] & 3) { d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w; }
            else *(float4*)d = x;
        }
    };
    for (int i = tid; i < n; i += kTabThreads) {
        const int q = i / V1;
        nxs[i] = (unsigned short)ctx_next(c, q, i - q * V1);
    }
    for (int d = tid; d < C; d += kTabThreads) be[d] = 0.f;
    auto put = [&](int t, double A) __attribute__((always_inline)) {
        const size_t row = a.keep ? (size_t)b * (a.T + 1) + t : (size_t)b;
        for (int d = tid; d < C; d += kTabThreads) a.beta[row * C + d] = be[d];
        if (tid == 0) a.offb[row] = A;
    };
    double A = 0.0;
    const int lpr = a.lpr, l = tid & (lpr - 1);
    const int epl = (V1 + lpr - 1) / lpr, y0 = l * epl;
    if (steps > 0) {
        spread(I0());
        issue(I0(), 2);
    }
    __syncthreads();
    if (a.keep || steps == 0) put(L, 0.0);
    auto frame = [&](auto S, int k) __attribute__((always_inline)) {
        constexpr int Z = decltype(S)::value;
        float mx = LAST_NEG_INF;
        const int rpp = kTabThreads / lpr;
        for (int q0 = 0; q0 < C; q0 += rpp) {
            const int q = q0 + tid / lpr;
            float m = LAST_NEG_INF, s = 0.f;
            if (q < C) {
                const int e1 = min(V1, y0 + epl);
                for (int y = y0; y < e1; y += 4) {           // four arcs at a time: one rescaling of the sum each
                    float x[4], mn = m;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = q * V1 + min(y + i, e1 - 1);
                        x[i] = tile[e] + be[nxs[e]];
                        if (y + i >= e1) x[i] = LAST_NEG_INF;
                        mn = fmaxf(mn, x[i]);
                    }
                    const float mm = mn == LAST_NEG_INF ? 0.f : mn;
                    s *= tri_exp(m - mm);
#pragma unroll
                    for (int i = 0; i < 4; ++i) s += tri_exp(x[i] - mm);
                    m = mn;
                }
            }
            for (int o = 1; o < lpr; o <<= 1) {
                const float om = __shfl_xor(m, o, kWave), os = __shfl_xor(s, o, kWave);
                const float mn = fmaxf(m, om), mm = mn == LAST_NEG_INF ? 0.f : mn;
                s = s * tri_exp(m - mm) + os * tri_exp(om - mm);
                m = mn;
            }
            const float x = ln_sum(m, s);
            if (q < C && l == 0) bc[q] = x;
            mx = fmaxf(mx, q < C ? x : LAST_NEG_INF);
        }
        mx = tab_block_max(mx, red);
        if (mx == LAST_NEG_INF) mx = 0.f;
        A += (double)mx;
        for (int d = tid; d < C; d += kTabThreads) be[d] = bc[d] - mx;
        if (a.keep || k + 1 == steps) put(L - 1 - k, A);
        spread(std::integral_constant<int, Z ^ 1>());
        issue(std::integral_constant<int, Z ^ 1>(), k + 3);
        lds_only_barrier();
    };
    for (int k = 0; k < steps; k += 2) {
        frame(I0(), k);
        if (k + 1 < steps) frame(I1(), k + 1);
    }
}

}  // namespace last
