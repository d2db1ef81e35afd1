// Arc marginals (Eq. 1 of arXiv 2304.13134) of the complete lattice from stored
// state vectors, for any context dependency: the whole chip streams over the
// frames, nothing is serial.
//   alpha, beta [B][T+1][C] base-2 logs, relative to the float64 offsets
//   offa, offb  [B][T+1];  D2 [B] base-2 log of the partition sum
//   dw[b][t][q][y] (+)= scale 2^(alpha_t[q] + w log2 e + beta_{t+1}[next(q,y)] + (offa_t + offb_{t+1} - D2))
// LINEAR: alpha, beta are linear relative to 2^offset and dw (+)= scale alpha 2^(w log2 e + offsets - D2) beta.
// There an entry more than 2^126 below the largest of its frame is zero; the marginal it would have had is below
// 2^-46 as long as the product of the frame's three maxima is below 2^80, and beyond that the item is
// flagged (kItemRange) and the exponent capped so that it stays finite (kMgExpCap).
// Bound: HBM, 4 bytes read and 4 written per arc.  A workgroup takes a stretch of rows of one frame, keeps
// its two state vectors in LDS (the row offset of the destinations with them) and goes through the stretch with
// 16-byte accesses on 16-byte boundaries of memory; rows are V+1 floats, so a piece may span rows.
#pragma once
#include "cluster_kernels.hpp"
#include "common.hpp"

namespace last {

constexpr int kMgThreads = 256;
constexpr float kMgRangeBits = 80.f;
// The forward weights are sums of at most 97 products below 2 each, times 2^(fraction) <= 2^(1/2): below 2^8.2; 2^f with
// |f| <= 1/2 adds half a bit and the backward weights, below 2, one: with this cap every product stays below 2^127.
constexpr float kMgExpCap = 117.f;
constexpr float kLog2eLow = 1.925963033500e-8f;      // log2 e - (float)log2 e
constexpr int kMgChunk = 32768;              // arcs of a workgroup, about

// grid (stretches, frames t0 ..., items).  ORDER 1, 2: closed form; 0: any context (badtab: flag of a bad next-state
// table, may be null).  skip: items whose marginals have been written already (may be null).
// LDS: float[C] alpha + exponent | float[C] beta.
template <int ORDER, bool ACC, bool LINEAR>
__global__ __launch_bounds__(kMgThreads) void dense_marginals_kernel(
    const float* __restrict__ w, const int* __restrict__ len, Ctx c, int T, int t0, int rows,
    const float* __restrict__ alpha, const float* __restrict__ beta, const double* __restrict__ offa,
    const double* __restrict__ offb, const double* __restrict__ D2, float* __restrict__ dw, float scale,
    const int* __restrict__ badtab, const int* __restrict__ skip, int* __restrict__ item_status)
{
    extern __shared__ float mg_s[];
    __shared__ float red[3][kMgThreads / kWave];
    float* al = mg_s;
    float* be = mg_s + c.C;
    const int t = t0 + blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int q0 = blockIdx.x * rows, q1 = min(q0 + rows, c.C);
    const size_t first = (((size_t)b * T + t) * c.C + q0) * c.V1;
    const int n = (q1 - q0) * c.V1;
    if (skip && skip[b] != 0) return;
    const int L = len[b];
    float* g = dw + first;
    const float* wt = w + first;
    // pieces of four that start on a 16-byte boundary of dw; up to three arcs before them
    const int lead = min((int)((4 - ((size_t)g >> 2)) & 3), n);
    const int n4 = (n - lead) / 4;
    if (L < 0 || L > T || t >= L || (ORDER == 0 && badtab && badtab[0] != 0)) {
        if (ACC) return;
        for (int i = tid; i < n4; i += kMgThreads) *(float4*)(g + lead + 4 * i) = make_float4(0.f, 0.f, 0.f, 0.f);
        if (tid < lead) g[tid] = 0.f;
        for (int i = lead + 4 * n4 + tid; i < n; i += kMgThreads) g[i] = 0.f;
        return;
    }
    float K, amax = 0.f, bmax = 0.f, wmax = LAST_NEG_INF;
    {
        const size_t ra = (size_t)b * (T + 1) + t;
        const double d2 = D2[b];                      // (-inf: no path, every product below is zero)
        const double kd = d2 == (double)LAST_NEG_INF ? 0.0 : offa[ra] + offb[ra + 1] - d2;
        // linear: the whole part goes into the exponent of 2^w, the fraction into the forward weights
        K = LINEAR ? (float)rint(fmin(fmax(kd, -1.0e9), 1.0e9)) : (float)kd;
        const float scaleK = LINEAR ? fast_exp2((float)(kd - (double)K)) : 1.f;
        for (int q = tid; q < c.C; q += kMgThreads) {
            const float x = alpha[ra * c.C + q], y = beta[(ra + 1) * c.C + q];
            if (LINEAR) {
                al[q] = x * scaleK;
                amax = fmaxf(amax, x);
                bmax = fmaxf(bmax, y);
            } else if (q >= q0 && q < q1) {
                al[q] = x + K;
            }
            be[q] = y;
        }
    }
    __syncthreads();
    auto arc = [&](int q, int y, float x) __attribute__((always_inline)) {
        int d = q;
        if (y > 0) {
            if (ORDER == 1) d = y;
            else if (ORDER == 2) d = (q == 0 ? 0 : ((q - 1) % c.V + 1) * c.V) + y;
            else d = ctx_next(c, q, y);
        }
        if (LINEAR) {
            wmax = fmaxf(wmax, x);
            // 2^(x log2 e + K) with the argument of exp2 reduced to [-1/2, 1/2]: its rounding would otherwise be
            // the largest error of a marginal
            const float y = fmaf(x, kLog2e, K), h = rintf(x * kLog2e);
            const float f = fmaf(x, kLog2eLow, fmaf(x, kLog2e, -h));
            const float e = y > -200.f ? __builtin_ldexpf(fast_exp2(f), (int)fminf(h + K, kMgExpCap)) : 0.f;
            return scale * (al[q] * e * be[d]);
        }
        return scale * fast_exp2(fmaf(x, kLog2e, al[q] + be[d]));
    };
    for (int i = tid; i < n4; i += kMgThreads) {
        const int e = lead + 4 * i;
        struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
        const f4 x = *(const f4*)(wt + e);
        int q = q0 + e / c.V1, y = e - (q - q0) * c.V1;
        float o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o[k] = arc(q, y, x.v[k]);
            const bool wrap = ++y == c.V1;
            q += wrap;
            y = wrap ? 0 : y;
        }
        float4* p = (float4*)(g + e);
        if (ACC) {
            const float4 old = *p;
            *p = make_float4(old.x + o[0], old.y + o[1], old.z + o[2], old.w + o[3]);
        } else {
            *p = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
    const int rest = n - lead - 4 * n4;
    if (tid < lead + rest) {
        const int e = tid < lead ? tid : lead + 4 * n4 + (tid - lead);
        const int q = q0 + e / c.V1, y = e - (q - q0) * c.V1;
        const float o = arc(q, y, wt[e]);
        if (ACC) g[e] += o; else g[e] = o;
    }
    if (LINEAR && item_status) {
        const int wv = tid / kWave;
        amax = wave_max(amax);
        bmax = wave_max(bmax);
        wmax = wave_max(wmax);
        if ((tid & (kWave - 1)) == 0) { red[0][wv] = amax; red[1][wv] = bmax; red[2][wv] = wmax; }
        __syncthreads();
        if (tid == 0) {
            for (int k = 1; k < kMgThreads / kWave; ++k) {
                amax = fmaxf(amax, red[0][k]);
                bmax = fmaxf(bmax, red[1][k]);
                wmax = fmaxf(wmax, red[2][k]);
            }
            if (amax > 0.f && bmax > 0.f && K + wmax * kLog2e + __builtin_amdgcn_logf(amax) + __builtin_amdgcn_logf(bmax) > kMgRangeBits)
                atomicMax(item_status + b, (int)kItemRange);
        }
    }
}

}  // namespace last
