// Arc marginals (Eq. 1 of arXiv 2304.13134) of the complete lattice from stored
// state vectors, for any context dependency: the whole chip streams over the
// frames, nothing is serial.
//   alpha, beta [B][T+1][C] natural logs, relative to the float64 offsets
//   offa, offb  [B][T+1];  D2 [B] log of the partition sum
//   dw[b][t][q][y] (+)= scale exp(alpha_t[q] + w + beta_{t+1}[next(q,y)] + offa_t + offb_{t+1}) / Z_{t+1}
// with Z_{t+1} = sum_q exp(alpha_{t+1}[q] + beta_{t+1}[q] + offsets), formed here.  It is the partition sum, but from
// the two vectors at hand: what the roundings of some hundred frames have moved the vectors by
// as a whole is in the numerator and in Z alike.  Divided by exp(D2), which has the roundings of the forward pass, it
// stayed in the marginals (their relative error together, against 64 bits, 61 frames, sigma 1.5: 5 states 2.7e-7 against
// 0.8e-7, a table of 200 states with 12 labels 1.2e-6 against 2.1e-7).  One more vector is read for each stretch of
// rows, 1 to 3 % of a call (loss at 8 items, 300 frames, 32 labels of order 2 0.737 -> 0.747 ms).
// LINEAR (bigram_kernels.hpp): alpha, beta are linear relative to 2^offset, offsets and D2 in base 2, and dw (+)= scale
// alpha 2^(w log2 e) beta 2^offsets / Z.  There an entry more than 2^126 below the largest of its frame may be zero; the
// marginal it would have had is below 2^-46 as long as the product of the frame's three maxima is below 2^80 Z,
// and beyond that the item is flagged (kItemRange).  It is flagged, too, where Z is not the partition sum: then one of the
// directions has lost a part of it.
// Bound: HBM, 4 bytes read and 4 written per arc.  A workgroup takes a stretch of rows of one frame, keeps
// its two state vectors in LDS (the row offset of the destinations with them) and goes through the stretch with
// 16-byte accesses on 16-byte boundaries of memory; rows are V+1 floats, so a piece may span rows.
#pragma once
#include "cluster_kernels.hpp"
#include "common.hpp"
#include "trigram_kernels.hpp"

namespace last {

constexpr int kMgThreads = 256;
constexpr float kMgRangeBits = 80.f;
// difference of two logarithms of the partition sum that no rounding makes: this much, and per frame
constexpr double kMgLostBits = 0.01, kMgLostBitsPerFrame = 1.0e-7;
constexpr int kMgAlphaExp = 65, kMgBetaExp = 59;      // alpha is below 2^127, beta below 2^120: taken down for their product
constexpr float kMgMax = 1.8e19f;            // 2^64: no marginal exceeds 1 but those of items that are flagged
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
    __shared__ double redz[kMgThreads / kWave];
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
    float K = 0.f, amax = 0.f, bmax = 0.f, wmax = LAST_NEG_INF, sc = scale;
    bool lost = false;
    const size_t ra = (size_t)b * (T + 1) + t;
    const int wv = tid / kWave;
    if (LINEAR) {
        double z = 0.0;
        for (int q = tid; q < c.C; q += kMgThreads) {
            const float x = __builtin_ldexpf(alpha[ra * c.C + q], -kMgAlphaExp);
            const float y = __builtin_ldexpf(beta[(ra + 1) * c.C + q], -kMgBetaExp);
            z += (double)alpha[(ra + 1) * c.C + q] * (double)y;
            al[q] = x;
            be[q] = y;
            amax = fmaxf(amax, x);
            bmax = fmaxf(bmax, y);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
        if ((tid & (kWave - 1)) == 0) redz[wv] = z;
        __syncthreads();
        z = redz[0];
#pragma unroll
        for (int k = 1; k < kMgThreads / kWave; ++k) z += redz[k];
        // 1 / Z: the exponent goes into that of 2^w (offsets are whole numbers), the mantissa into the scale
        const double d2 = D2[b];                  // (-inf: no path, every product below is zero)
        if (z > 0.0) {
            int e;
            const double m = frexp(z, &e);        // in [1/2, 1)
            K = (float)(offa[ra] - offa[ra + 1] - (double)(e - kMgAlphaExp));          // (z has beta's factor, too)
            sc = scale / (float)m;
            lost = !(fabs(offa[ra + 1] + offb[ra + 1] + (double)((float)(e + kMgBetaExp) + __builtin_amdgcn_logf((float)m)) - d2)
                     < kMgLostBits + kMgLostBitsPerFrame * L);
        } else {
            lost = d2 != (double)LAST_NEG_INF;
        }
    } else {
        float m = LAST_NEG_INF, z = 0.f;
        for (int q = tid; q < c.C; q += kMgThreads) {
            const float x = alpha[ra * c.C + q], y = beta[(ra + 1) * c.C + q];
            const float a1 = alpha[(ra + 1) * c.C + q], v = a1 == LAST_NEG_INF ? a1 : a1 + y;
            const float n = fmaxf(m, v), nn = n == LAST_NEG_INF ? 0.f : n;
            z = fmaf(z, tri_exp(m - nn), tri_exp(v - nn));
            m = n;
            if (q >= q0 && q < q1) al[q] = x;
            be[q] = y;
        }
        const float mw = wave_max_dpp(m), mn = mw == LAST_NEG_INF ? 0.f : mw;
        z = wave_sum_dpp(z * tri_exp(m - mn));
        if ((tid & (kWave - 1)) == 0) { red[0][wv] = mw; red[1][wv] = z; }
        __syncthreads();
        float M = red[0][0];
#pragma unroll
        for (int k = 1; k < kMgThreads / kWave; ++k) M = fmaxf(M, red[0][k]);
        const float MM = M == LAST_NEG_INF ? 0.f : M;     // (no path: every exponential below is zero)
        z = 0.f;
#pragma unroll
        for (int k = 0; k < kMgThreads / kWave; ++k) z += red[1][k] * tri_exp(red[0][k] - MM);
        sc = M == LAST_NEG_INF ? scale : scale / z;
        const double kd = offa[ra] - offa[ra + 1] - (double)MM;
        for (int q = q0 + tid; q < q1; q += kMgThreads) al[q] = (float)((double)al[q] + kd);
    }
    __syncthreads();
    // ORDER 2: the label arcs of state q lead to the states after row_base(q), those of q + 1 to V states further on (after
    // the last label from the first again)
    auto row_base = [&](int q) __attribute__((always_inline)) { return ORDER == 2 && q > 0 ? ((q - 1) % c.V + 1) * c.V : 0; };
    auto next_base = [&](int base) __attribute__((always_inline)) { return base == c.V * c.V ? c.V : base + c.V; };
    auto arc = [&](int q, int y, int base, float x) __attribute__((always_inline)) {
        int d = q;
        if (y > 0) {
            if (ORDER == 1) d = y;
            else if (ORDER == 2) d = base + y;
            else d = ctx_next(c, q, y);
        }
        if (LINEAR) {
            wmax = fmaxf(wmax, x);
            // 2^(x log2 e + K) with the argument of exp2 reduced to [-1/2, 1/2]: its rounding would otherwise be
            // the largest error of a marginal
            const float y = fmaf(x, kLog2e, K), h = rintf(x * kLog2e);
            const float f = fmaf(x, kLog2eLow, fmaf(x, kLog2e, -h));
            const float e = y > -300.f ? fast_exp2(f) : 0.f;               // (the product of the vectors is below 2^123)
            return sc * fminf(__builtin_ldexpf(al[q] * be[d] * e, (int)(h + K)), kMgMax);
        }
        // (an arc out of an unreachable state does not count, whatever its weight)
        return al[q] == LAST_NEG_INF ? 0.f : sc * tri_exp(al[q] + be[d] + x);
    };
    for (int i = tid; i < n4; i += kMgThreads) {
        const int e = lead + 4 * i;
        struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
        const f4 x = *(const f4*)(wt + e);
        int q = q0 + e / c.V1, y = e - (q - q0) * c.V1;
        int base = row_base(q);
        float o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o[k] = arc(q, y, base, x.v[k]);
            const bool wrap = ++y == c.V1;
            q += wrap;
            y = wrap ? 0 : y;
            if (ORDER == 2) base = wrap ? next_base(base) : base;
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
        const float o = arc(q, y, row_base(q), wt[e]);
        if (ACC) g[e] += o; else g[e] = o;
    }
    if (LINEAR && item_status) {
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
            if (lost || (amax > 0.f && bmax > 0.f
                         && K + wmax * kLog2e + __builtin_amdgcn_logf(amax) + __builtin_amdgcn_logf(bmax) > kMgRangeBits))
                atomicMax(item_status + b, (int)kItemRange);
        }
    }
}

}  // namespace last
