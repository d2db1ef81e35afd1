// The recursions for a next-state table in the log semiring, both directions at once (one workgroup per item and
// direction), for frames of 3072 to 8192 arcs and up to 1024 states; other ones, and items of few frames, take table_chain_kernels.hpp.
//
// Both directions are the same sum over lists of arcs: of those that lead to a state (forward), of those that leave it
// (backward),
//     new[s] = log sum_{arcs i of s} exp(w[arc_i] + old[other_i]).
// The lists are made once an item (forward: counted, laid out by state and put in the order of the arcs, so that sums do not depend
// on timing), and a lane keeps its share of one, 16 bits of arc and 16 of state each, in registers for all frames; what is
// longer than 12 arcs a lane is read from LDS.  A frame is two LDS reads and an exponential an arc, a reduction over the lanes
// of a row and one barrier.  Pushing arcs with LDS atomics (table_chain_kernels.hpp) took four barriers and two atomics an
// arc.  Weights go through LDS, two frames of them, requested two frames ahead.
// Natural logs relative to a float64 offset per frame.  The offset of a frame is what its largest entry will be if it grows as it
// did in the frame before, so that no frame waits for its own maximum.
// Bound: vector ALU and LDS latency of a frame's chain.  Measured (8 items, 120 to 200 frames, 585 states, 8 labels): both directions
// 1.7 us a frame instead of 2.5, the loss with gradient 0.39 instead of 0.54 ms.
#pragma once
#include "table_chain_kernels.hpp"

namespace last {

constexpr int kTpThreads = 1024;
constexpr int kTpMinArcs = 3072, kTpMaxArcs = 8192, kTpMaxStates = 1024, kTpMinFrames = 48;
constexpr int kTpArcs = 12;          // arcs of a lane in registers
constexpr int kTpPieces = kTpMaxArcs / 4 / kTpThreads;

__host__ __device__ inline size_t tp_lds(int C, int V1)
{
    const size_t n = (size_t)C * V1, pad = (n + 8) & ~(size_t)3;
    return (2 * pad + n + 2 * (size_t)C + 2 * (size_t)C + 2 + 64) * sizeof(float);
}

// over the LPR lanes of a row
template <bool MAX>
__device__ __forceinline__ float tp_row(float x, int lpr)
{
    auto op = [](float a, float b) __attribute__((always_inline)) { return MAX ? fmaxf(a, b) : a + b; };
    if (lpr > 1) x = op(x, dpp_f<0xB1>(x, x));                       // quad_perm 1,0,3,2
    if (lpr > 2) x = op(x, dpp_f<0x4E>(x, x));                       // quad_perm 2,3,0,1
    if (lpr > 4) x = op(x, dpp_f<0x141>(x, x));                      // row_half_mirror
    if (lpr > 8) x = op(x, dpp_f<0x140>(x, x));                      // row_mirror
    for (int o = 16; o < lpr; o <<= 1) x = op(x, __shfl_xor(x, o, kWave));
    return x;
}

template <bool back>
__device__ __forceinline__ void table_pull(const TabArgs& a, const Ctx& c)
{
    extern __shared__ __align__(16) float tp_s[];
    constexpr int NT = kTpThreads, NW = NT / kWave, NQ = kTpPieces;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = c.C, V1 = c.V1, n = C * V1, pad = (n + 8) & ~3;
    const int L = a.len[b];
    const bool badtab = a.bad && a.bad[0] != 0;
    if (L < 0 || L > a.T || badtab) {
        if (a.keep && !back && tid == 0) {
            a.dist[b] = __builtin_nanf("");
            a.D2[b] = __builtin_nan("");
            if (a.item_status) a.item_status[b] = badtab ? kItemBadTable : kItemBadLength;
        }
        return;
    }
    const int low = a.keep ? 1 : L / 2;
    const int steps = back ? max(L - low, 0) : a.keep ? L : L / 2;
    const float* wi = a.w + (size_t)b * a.T * n;
    float* const tile = tp_s;                               // [2][pad] weights; [n]: a weight that is none
    unsigned* const list = (unsigned*)(tile + 2 * pad);     // [n] arc | other state << 16, by state
    float* const vec = (float*)(list + n);                  // [2][C]
    int* const start = (int*)(vec + 2 * C);                 // [C + 1] first arc of a state
    int* const cnt = start + C + 1;                         // [C]
    float* const red = (float*)(cnt + C + 1);               // [2][NW]
    __shared__ int sums[NW];

    // pieces of a thread, as in table_chain_kernel
    int pf[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) pf[j] = min(4 * (tid + NT * j), n - 4);
    float4 raw[2][NQ];
    auto issue = [&](auto S, int k) __attribute__((always_inline)) {
        const int t = back ? max(L - 1 - k, 0) : min(k, max(L - 1, 0));
        const buf_t rs = make_buf(wi + (size_t)t * n, 4u * (unsigned)n);
#pragma unroll
        for (int j = 0; j < NQ; ++j) raw[decltype(S)::value][j] = tri_load4(rs, 4u * (unsigned)pf[j], 0);
    };
    auto spread = [&](auto S) __attribute__((always_inline)) {       // (pieces past the frame write its last one again)
        constexpr int Z = decltype(S)::value;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            float* d = tile + Z * pad + pf[j];
            const float4 x = raw[Z][j];
            if (pf[j] & 3) { d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w; }
            else *(float4*)d = x;
        }
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    if (steps > 0) {
        issue(I0(), 0);
        issue(I1(), 1);
    }

    // the lists
    if (back) {
        for (int i = tid; i < n; i += NT) {
            const int q = i / V1;
            list[i] = (unsigned)i | (unsigned)ctx_next(c, q, i - q * V1) << 16;
        }
        for (int d = tid; d <= C; d += NT) start[d] = d * V1;
    } else {
        unsigned* const any = (unsigned*)tile;              // arcs of a state in any order (the tiles are not in use yet)
        constexpr int PA = kTpMaxArcs / NT;
        unsigned arcs[PA];                                  // arc | state it leads to << 16
        if (tid < C) cnt[tid] = 0;
#pragma unroll
        for (int j = 0; j < PA; ++j) {
            arcs[j] = 0;
            if (NT * j >= n) continue;
            const int i = min(tid + NT * j, n - 1), q = i / V1;
            arcs[j] = (unsigned)i | (unsigned)ctx_next(c, q, i - q * V1) << 16;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PA; ++j)
            if (tid + NT * j < n) atomicAdd(&cnt[arcs[j] >> 16], 1);
        __syncthreads();
        const int own = tid < C ? cnt[tid] : 0;             // (C <= NT)
        int sum = own;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int x = __shfl_up(sum, o, kWave);
            sum += lane >= o ? x : 0;
        }
        if (lane == kWave - 1) sums[wave] = sum;
        __syncthreads();
        for (int k = 0; k < wave; ++k) sum += sums[k];
        if (tid < C) {
            start[tid + 1] = sum;
            cnt[tid] = sum - own;
            if (tid == 0) start[0] = 0;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PA; ++j)
            if (tid + NT * j < n) any[atomicAdd(&cnt[arcs[j] >> 16], 1)] = arcs[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PA; ++j) {
            if (tid + NT * j >= n) continue;
            const unsigned arc = arcs[j] & 0xffffu, d = arcs[j] >> 16;
            int place = start[d];
            for (int k = start[d]; k < start[d + 1]; ++k) place += (any[k] & 0xffffu) < arc;
            list[place] = arc | (arc / (unsigned)V1) << 16;
        }
    }
    for (int d = tid; d < C; d += NT) vec[d] = back || d == 0 ? 0.f : LAST_NEG_INF;
    __syncthreads();
    if (tid < 8) {
        if (n + tid < pad) tile[n + tid] = tile[pad + n + tid] = LAST_NEG_INF;
    }

    // this lane's share of its row
    const int lpr = a.lpr, l = tid & (lpr - 1), row = tid / lpr;
    const bool mine = row < C;
    const int first = mine ? start[row] + l : 0, last = mine ? start[row + 1] : 0;
    unsigned wOff[kTpArcs], oOff[kTpArcs];                  // bytes
#pragma unroll
    for (int i = 0; i < kTpArcs; ++i) {
        const unsigned e = first + lpr * i < last ? list[first + lpr * i] : (unsigned)n;
        wOff[i] = 4u * (e & 0xffffu);
        oOff[i] = 4u * (e >> 16);
    }
    const unsigned at = mine && l == 0 ? 4u * (unsigned)row : 0xfffffff0u;
    const int share = max(0, (last - first + lpr - 1) / lpr);
    const int most = wave_max_dpp(share);                   // of the wave
    __syncthreads();                                        // (the lists' temporary is done with)

    double A = 0.0;
    float o = 0.f, M = 0.f, before = 0.f;                   // offset step of the frame before, its largest entry, that of the one before
    auto put = [&](float* base, double* off, int t, const float* v) __attribute__((always_inline)) {
        const size_t r = a.keep ? (size_t)b * (a.T + 1) + t : (size_t)b;
        for (int d = tid; d < C; d += NT) base[r * C + d] = v[d];
        if (tid == 0) off[r] = A;
    };
    if (steps > 0) {
        spread(I0());
        issue(I0(), 2);
    }
    __syncthreads();
    if (back ? a.keep || steps == 0 : a.keep || steps == 0) put(back ? a.beta : a.alpha, back ? a.offb : a.offa, back ? L : 0, vec);
    auto frame = [&](auto S, int k) __attribute__((always_inline)) {
        constexpr int Z = decltype(S)::value;
        const float* const w = tile + Z * pad;
        const float* const old = vec + Z * C;
        float* const now = vec + (Z ^ 1) * C;
        // the largest entry of the vector at hand
        if (k > 0) {
            float x = red[Z * NW];
#pragma unroll
            for (int i = 1; i < NW; ++i) x = fmaxf(x, red[Z * NW + i]);
            before = M;
            M = x;
        }
        const float grown = M + o - before;
        o = M == LAST_NEG_INF || before == LAST_NEG_INF ? 0.f : k > 0 ? M + grown : 0.f;
        // (an arc out of an unreachable state does not count, whatever its weight)
        auto score = [&](unsigned wo, unsigned oo) __attribute__((always_inline)) {
            const float x = *(const float*)((const char*)old + oo), y = *(const float*)((const char*)w + wo);
            return !back && x == LAST_NEG_INF ? x : y + x;
        };
        auto more = [&](unsigned e) __attribute__((always_inline)) { return score(4u * (e & 0xffffu), 4u * (e >> 16)); };
        float v[kTpArcs], m = LAST_NEG_INF;
        // (four arcs at a time; none beyond the longest share of the wave)
#pragma unroll
        for (int i0 = 0; i0 < kTpArcs; i0 += 4)
            if (i0 < most) {
#pragma unroll
                for (int i = i0; i < i0 + 4; ++i) {
                    v[i] = score(wOff[i], oOff[i]);
                    m = fmaxf(m, v[i]);
                }
            }
        for (int i = first + lpr * kTpArcs; i < last; i += lpr) m = fmaxf(m, more(list[i]));
        m = tp_row<true>(m, lpr);
        const float mm = m == LAST_NEG_INF ? 0.f : m;
        float z = 0.f;
#pragma unroll
        for (int i0 = 0; i0 < kTpArcs; i0 += 4)
            if (i0 < most) {
#pragma unroll
                for (int i = i0; i < i0 + 4; ++i) z += tri_exp(v[i] - mm);
            }
        double rest = 0.0;                                  // (there may be thousands)
        for (int i = first + lpr * kTpArcs; i < last; i += lpr) rest += (double)tri_exp(more(list[i]) - mm);
        z = tp_row<false>(z + (float)rest, lpr);
        const float x = mine ? ln_sum(m, z) - o : LAST_NEG_INF;
        if (mine && l == 0) now[row] = x;
        const float top = wave_max_dpp(x);
        if (lane == 0) red[(Z ^ 1) * NW + wave] = top;
        const bool live = k < steps;                        // (frames go in pairs, so that the waits are counted; one too many leaves no trace)
        A += live ? (double)o : 0.0;
        // (stores on every path, dropped by the range check: the waits for the weights are counted)
        const bool stored = a.keep && live;
        const size_t r = stored ? (size_t)b * (a.T + 1) + (back ? L - 1 - k : k + 1) : 0;
        buf_store(x, make_buf((back ? a.beta : a.alpha) + r * C, stored ? 4u * (unsigned)C : 0u), at, 0);
        nw_store64(A, make_buf((back ? a.offb : a.offa) + r, stored ? 8u : 0u), tid == 0 ? 0u : 0xfffffff0u, 0);
        spread(std::integral_constant<int, Z ^ 1>());
        issue(std::integral_constant<int, Z ^ 1>(), k + 3);
        lds_only_barrier();
    };
    for (int k = 0; k < steps; k += 2) {
        frame(I0(), k);
        frame(I1(), k + 1);
    }
    const float* const end = vec + (steps & 1) * C;
    if (!a.keep) {
        if (steps > 0) put(back ? a.beta : a.alpha, back ? a.offb : a.offa, 0, end);
        return;
    }
    if (back) return;
    // all states of the last frame are final with weight 0
    float mx = LAST_NEG_INF;
    if (tid < C) mx = end[tid];
    const float keep = mx;
    mx = wave_max_dpp(mx);
    __syncthreads();
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0];
    for (int i = 1; i < NW; ++i) mx = fmaxf(mx, red[i]);
    const float mm = mx == LAST_NEG_INF ? 0.f : mx;
    double z = tid < C ? (double)tri_exp(keep - mm) : 0.0;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) z += __shfl_xor(z, s, kWave);
    double* const redd = (double*)tile;
    if (lane == 0) redd[wave] = z;
    __syncthreads();
    if (tid == 0) {
        z = 0.0;
        for (int i = 0; i < NW; ++i) z += redd[i];
        const double d2 = mx == LAST_NEG_INF ? (double)LAST_NEG_INF : A + (double)mm + log(z);
        a.D2[b] = d2;
        a.dist[b] = (float)d2;
        if (a.item_status) a.item_status[b] = kItemOk;
    }
}

__global__ __launch_bounds__(kTpThreads) void table_pull_kernel(TabArgs a, Ctx c)
{
    if (blockIdx.y == 1) table_pull<true>(a, c);
    else table_pull<false>(a, c);
}

}  // namespace last
