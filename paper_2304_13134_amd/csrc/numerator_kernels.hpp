// Numerator of the globally normalised loss: the complete lattice intersected
// with the reference label string, and the log-semiring shortest distance on
// the resulting (t, u) grid (arXiv 2304.13134, Section 2.1; Table 1 "GNAT,
// intersected": O(TU) states and arcs, small enough to store).
//
// Three stages, all on the caller's stream:
//   1. gather   : the 2 arc weights leaving every (t, u) are pulled out of the
//                 dense tensor into a compact [B][T][U1][2] array (fully
//                 parallel, it is the only stage that touches the big tensor);
//   2. recursion: per item one workgroup runs the forward weights and a second
//                 one the backward weights, frame-serial, state-parallel;
//   3. scatter  : arc marginals exp(a + w + b' - N) are added onto the arcs of
//                 the complete lattice they ride on.
// The locally normalised variant (Section 2.1: a model like RNN-T is the same
// intersection followed by a shortest distance, with the arcs leaving each state
// normalised; Table 1, first row) adds to the gather the log-sum-exp lz of the
// V+1 arcs leaving (t, ctx(u)), subtracts it in the recursion, and its scatter
// writes d/dw = marginals - (occupancy of the state) * softmax(row), row by row.
// Grid values are kept in float64 (they reach several thousand and feed an
// exponent that must be good to 1e-6); the transcendental part of each
// log-add-exp has an O(1) argument and is evaluated in float32.
#pragma once
#include "cluster_kernels.hpp"
#include "common.hpp"

namespace last {

// context state after the first u reference labels
__device__ __forceinline__ int ref_context(const Ctx& c, const int* __restrict__ r, int u)
{
    if (u == 0) return 0;
    if (c.order == 1 || u == 1) return r[u - 1];
    return 1 + c.V + (r[u - 2] - 1) * c.V + (r[u - 1] - 1);
}

__device__ __forceinline__ int clamp_label(int y, int V) { return y < 1 ? 1 : (y > V ? V : y); }

// status [B]: 0 ok, or the item_status code of the first problem found.
// ctxs [B][U1]: context state after the first u reference labels (-1 past U).
// link [B][U1][2]: [0] = the next u' > u with the same context (-1: none), [1] = 1 when no
// u' < u has the same context (u heads its chain).  Cells of one chain ride on the same rows
// of the complete lattice.
// Bound: latency (one workgroup an item, in front of the gather).  The contexts stay in LDS, a wave compares 64 of them at a time,
// and a next-state table of up to kNcTable entries is walked in LDS: 150 labels 25 -> 9 us, 60 labels 13 -> 4.7 us, 80 labels through a table
// of 585 x 8 entries 27 -> 12 us, against a thread per cell that looked through global memory and a walk of
// dependent loads.  LDS: int[U1] contexts (fewer than 4096 labels), then int[C V] the table (table_lds).
constexpr int kNcThreads = 1024;        // at most; whole waves
constexpr int kNcTable = 12032;         // 47 KiB, beside the 16 of the contexts
__global__ __launch_bounds__(kNcThreads) void num_check_kernel(const int* __restrict__ len, const int* __restrict__ refs,
                                 const int* __restrict__ ulen, Ctx c, int T, int Umax,
                                 int* __restrict__ status, int* __restrict__ ctxs,
                                 int* __restrict__ link, const int* __restrict__ badtab, int table_lds)
{
    extern __shared__ int nc_s[];
    __shared__ int bad;
    const int b = blockIdx.x, tid = threadIdx.x;
    const int U1 = Umax + 1;
    if (tid == 0) bad = 0;
    const int L = len[b], U = ulen[b];
    const bool wrong = badtab && badtab[0];
    const int* r = refs + (size_t)b * Umax;
    int* cx = ctxs + (size_t)b * U1;
    int* q_s = nc_s;
    int* nx_s = nc_s + U1;
    if (table_lds)
        for (int i = tid; i < c.C * c.V; i += blockDim.x) nx_s[i] = min((unsigned)c.nx[i], (unsigned)(c.C - 1));
    int code = kItemOk;
    __syncthreads();
    if (wrong) code = kItemBadTable;
    else if (L < 0 || L > T) code = kItemBadLength;
    else if (U < 0 || U > Umax) code = kItemBadRefLength;
    else {
        for (int u = tid; u < U; u += blockDim.x) {
            const int y = r[u];
            if (y < 1 || y > c.V) atomicOr(&bad, 1);
            else if (c.order == 0) q_s[u + 1] = y;        // (labels, until the walk comes by)
        }
    }
    __syncthreads();
    if (code == kItemOk && bad) code = kItemBadLabel;
    if (code == kItemOk && U > L) code = kItemInfeasible;
    if (tid == 0) status[b] = code;
    if (code != kItemOk && code != kItemInfeasible) {
        for (int u = tid; u < U1; u += blockDim.x) cx[u] = -1;
        return;
    }
    if (c.order == 0) {
        // a general automaton has to be walked label by label
        if (tid == 0) {
            int q = 0;
            q_s[0] = 0;
            for (int u = 1; u <= U; ++u) {
                const int y = q_s[u];
                q = table_lds ? nx_s[q * c.V + y - 1] : ctx_next(c, q, y);
                q_s[u] = q;
            }
        }
        __syncthreads();
        for (int u = tid; u <= U; u += blockDim.x) cx[u] = q_s[u];
    } else {
        for (int u = tid; u <= U; u += blockDim.x) {
            const int q = ref_context(c, r, u);
            q_s[u] = q;
            cx[u] = q;
        }
    }
    for (int u = U + 1 + tid; u < U1; u += blockDim.x) cx[u] = -1;
    __syncthreads();
    int* lk = link + (size_t)b * U1 * 2;
    const int lane = tid & (kWave - 1);
    for (int u = tid / kWave; u < U1; u += blockDim.x / kWave) {        // (uniform in a wave)
        int nxt = -1, head = 1;
        if (u <= U) {
            const int q = q_s[u];
            for (int v0 = u + 1; v0 <= U; v0 += kWave) {
                const unsigned long long same = __ballot(v0 + lane <= U && q_s[min(v0 + lane, U)] == q);
                if (same) { nxt = v0 + __ffsll(same) - 1; break; }
            }
            for (int v0 = u - 1; v0 >= 0; v0 -= kWave)
                if (__any(v0 - lane >= 0 && q_s[max(v0 - lane, 0)] == q)) { head = 0; break; }
        } else {
            head = 0;
        }
        if (lane < 2) lk[2 * u + lane] = lane == 0 ? nxt : head;
    }
}

// wi[b][t][u][0] = w[b][t][ctx(u)][0]; wi[b][t][u][1] = w[b][t][ctx(u)][ref[u]] (u < U)
__global__ void num_gather_kernel(const float* __restrict__ w, const int* __restrict__ len,
                                  const int* __restrict__ refs, const int* __restrict__ ulen,
                                  const int* __restrict__ status, const int* __restrict__ ctxs,
                                  Ctx c, int T, int Umax, float2* __restrict__ wi)
{
    const int U1 = Umax + 1;
    const int b = blockIdx.z, t = blockIdx.y;
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= U1 || status[b] != kItemOk) return;
    const int L = len[b], U = ulen[b];
    if (t >= L || u > U) return;
    const int* r = refs + (size_t)b * Umax;
    const int q = ctxs[(size_t)b * U1 + u];
    const float* row = w + (((size_t)b * T + t) * c.C + q) * c.V1;
    float2 o;
    o.x = row[0];
    o.y = (u < U) ? row[r[u]] : LAST_NEG_INF;
    wi[((size_t)b * T + t) * U1 + u] = o;
}

// One row of V1 floats across the lanes of a wavefront in 16-byte pieces (rows are only 4-byte aligned): lane l
// holds pieces l, l + 64, ..; the last piece of the row ends with it, what it shares with the piece before does not count.
template <int QL>
struct NumRow {
    float w[QL][4];
};
template <int QL>
struct NumPieces {
    int at[QL];          // first column of the piece
    int skip[QL];        // leading columns that do not count (4: the whole piece)
    // c0: first column (a row of more than 256 QL weights goes by stretches of that many)
    __device__ __forceinline__ NumPieces(int V1, int lane, int c0 = 0)
    {
#pragma unroll
        for (int j = 0; j < QL; ++j) {
            const int c = c0 + 4 * (lane + kWave * j);
            at[j] = min(c, V1 - 4);
            skip[j] = min(c - at[j], 4);
        }
    }
};
template <int QL>
__device__ __forceinline__ NumRow<QL> num_load_row(const float* __restrict__ row, const NumPieces<QL>& p)
{
    struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
    NumRow<QL> r;
#pragma unroll
    for (int j = 0; j < QL; ++j) {
        const f4 x = *(const f4*)(row + p.at[j]);
#pragma unroll
        for (int k = 0; k < 4; ++k) r.w[j][k] = x.v[k];
    }
    return r;
}

// sum over the wave in float64, without LDS
template <int CTRL, int ROWS>
__device__ __forceinline__ double num_shifted(double x)      // 0 where no lane is behind
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double num_wave_sum(double x)
{
    x += num_shifted<0x111, 0xf>(x);
    x += num_shifted<0x112, 0xf>(x);
    x += num_shifted<0x114, 0xf>(x);
    x += num_shifted<0x118, 0xf>(x);
    x += num_shifted<0x142, 0xa>(x);
    x += num_shifted<0x143, 0xc>(x);
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, 63), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), 63);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// e^x for x <= 0, with the error of expf (2.6e-8 rms, 8e-8 at most): the argument of exp2 is reduced to [-1/2, 1/2] and what
// the product with log2 e is rounded by goes with it.  Below -150 it is 0: the reduction does not hold for masks of -1e10 (what a
// product is rounded by is no small number there), lowest values (the product is not finite) and -inf.  NaN stays NaN.
__device__ __forceinline__ float num_exp(float x)
{
#pragma clang fp contract(off)
    const float y = x < -150.f ? -150.f : x;
    const float p = y * kLog2e, h = rintf(p);
    const float f = (p - h) + fmaf(y, 1.925963033500e-8f, fmaf(y, kLog2e, -p));      // log2 e - (float)log2 e
    return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), (int)h);
}

// Locally normalised variant of the gather: a wavefront takes kNlFrames neighbouring frames of one u,
//   lz[b][t][u] = log sum_y exp w[b][t][ctx(u)][y],  wd[b][t][u] = w - lz of the two arcs (float64).
// Cells outside the cone that paths from (0,0) to (len, U) can visit get zeros without touching the
// weights (their forward or backward weight is -inf, whatever the arc weights).
// Bound: HBM, one row of the frame per cell.  Rows are read once, with 16-byte loads into registers, those of the
// wave's frames in flight together: B=16, T=500, V=256, 50 to 150 labels 0.58 -> 0.25 ms against one cell per
// wave whose row was read twice, 4 bytes a lane.  Rows of more than 512 weights (QL = 0) are read twice, in stretches
// of 256, the second time from cache.
constexpr int kNlFrames = 4;
template <int QL>
__global__ __launch_bounds__(256) void num_gather_local_kernel(
    const float* __restrict__ w, const int* __restrict__ len, const int* __restrict__ refs,
    const int* __restrict__ ulen, const int* __restrict__ status, const int* __restrict__ ctxs,
    Ctx c, int T, int Umax, double2* __restrict__ wd, double* __restrict__ lz)
{
    const int U1 = Umax + 1;
    const int b = blockIdx.z, t0 = blockIdx.y * kNlFrames;
    const int u = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (u >= U1 || status[b] != kItemOk) return;
    const int L = len[b], U = ulen[b];
    if (t0 >= L || u > U) return;
    const int q = ctxs[(size_t)b * U1 + u];
    const int y1 = u < U ? refs[(size_t)b * Umax + u] : 0;
    const size_t fr = (size_t)c.C * c.V1;
    const float* row0 = w + ((size_t)b * T * c.C + q) * c.V1;
    bool in[kNlFrames];
    float m[kNlFrames], w0[kNlFrames], w1[kNlFrames];
    double s[kNlFrames];                         // the lanes' sums are added up in float64
    auto lanes = [](double x) __attribute__((always_inline)) { return num_wave_sum(x); };
    auto one = [&](int i) __attribute__((always_inline)) {
        const int t = min(t0 + i, L - 1);
        return row0 + (size_t)t * fr;
    };
#pragma unroll
    for (int i = 0; i < kNlFrames; ++i) in[i] = t0 + i < L && u <= t0 + i && U - u <= L - (t0 + i);
    if (QL > 0) {
        constexpr int Q = QL > 0 ? QL : 1;
        const NumPieces<Q> p(c.V1, lane);
        NumRow<Q> r[kNlFrames];
#pragma unroll
        for (int i = 0; i < kNlFrames; ++i) {
            const float* row = one(in[i] ? i : 0);
            r[i] = num_load_row<Q>(row, p);
            w0[i] = row[0];
            w1[i] = row[y1];
        }
#pragma unroll
        for (int i = 0; i < kNlFrames; ++i) {
            m[i] = LAST_NEG_INF;
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) m[i] = fmaxf(m[i], r[i].w[j][k]);
            m[i] = wave_max_dpp(m[i]);
            const float mm = m[i] == LAST_NEG_INF ? 0.f : m[i];
            float si = 0.f;
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) si += k >= p.skip[j] ? num_exp(r[i].w[j][k] - mm) : 0.f;
            s[i] = lanes((double)si);
        }
    } else if (c.V1 >= 4) {
        float mi[kNlFrames], si[kNlFrames];
#pragma unroll
        for (int i = 0; i < kNlFrames; ++i) {
            const float* row = one(in[i] ? i : 0);
            mi[i] = LAST_NEG_INF;
            si[i] = 0.f;
            w0[i] = row[0];
            w1[i] = row[y1];
        }
        auto stretch = [&](int c0, auto&& f) __attribute__((always_inline)) {
            const NumPieces<1> p(c.V1, lane, c0);
            NumRow<1> r[kNlFrames];
#pragma unroll
            for (int i = 0; i < kNlFrames; ++i) r[i] = num_load_row<1>(one(in[i] ? i : 0), p);
#pragma unroll
            for (int i = 0; i < kNlFrames; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) f(i, r[i].w[0][k], k >= p.skip[0]);
        };
        for (int c0 = 0; c0 < c.V1; c0 += 4 * kWave)
            stretch(c0, [&](int i, float x, bool) __attribute__((always_inline)) { mi[i] = fmaxf(mi[i], x); });
#pragma unroll
        for (int i = 0; i < kNlFrames; ++i) {
            m[i] = wave_max_dpp(mi[i]);
            mi[i] = m[i] == LAST_NEG_INF ? 0.f : m[i];
        }
        for (int c0 = 0; c0 < c.V1; c0 += 4 * kWave)
            stretch(c0, [&](int i, float x, bool counts) __attribute__((always_inline)) { si[i] += counts ? num_exp(x - mi[i]) : 0.f; });
#pragma unroll
        for (int i = 0; i < kNlFrames; ++i) s[i] = lanes((double)si[i]);
    } else {
#pragma unroll 1
        for (int i = 0; i < kNlFrames; ++i) {
            const float* row = one(in[i] ? i : 0);
            float mi = LAST_NEG_INF, si = 0.f;
            for (int y = lane; y < c.V1; y += kWave) mi = fmaxf(mi, row[y]);
            mi = wave_max_dpp(mi);
            if (mi != LAST_NEG_INF)
                for (int y = lane; y < c.V1; y += kWave) si += expf(row[y] - mi);
            m[i] = mi;
            s[i] = lanes((double)si);
            w0[i] = row[0];
            w1[i] = row[y1];
        }
    }
    if (lane < kNlFrames && t0 + lane < L) {
        bool inl = in[0];
        float ml = m[0], w0l = w0[0], w1l = w1[0];
        double sl = s[0];
#pragma unroll
        for (int i = 1; i < kNlFrames; ++i)
            if (lane == i) { inl = in[i]; ml = m[i]; sl = s[i]; w0l = w0[i]; w1l = w1[i]; }
        const size_t cell = ((size_t)b * T + t0 + lane) * U1 + u;
        const double z = !inl ? 0.0 : ml == LAST_NEG_INF ? (double)LAST_NEG_INF : (double)ml + log(sl);
        lz[cell] = z;
        double2 o;
        o.x = inl ? (double)w0l - z : 0.0;
        o.y = inl ? (u < U ? (double)w1l - z : (double)LAST_NEG_INF) : 0.0;
        wd[cell] = o;
    }
}

// log(exp x + exp y): the large part m in float64, the correction log(1 + exp(lo - m)) in (0, log 2]
// with the hardware exp2 / log2 (absolute error of a few 1e-8, far below what feeds an exponent
// that must be good to 1e-6 after a few hundred frames)
__device__ __forceinline__ double log_add(double x, double y)
{
    const double m = x > y ? x : y;
    if (m == (double)LAST_NEG_INF) return m;
    const double lo = x > y ? y : x;
    const float d = (float)(lo - m);           // <= 0, -inf allowed
    return m + (double)__logf(1.f + __expf(d));
}

// grid (B, 2): blockIdx.y = 0 forward weights a[b][t][u], = 1 backward weights bk.
// Both arrays are [B][T+1][U1] float64; cells outside the reachable cone hold -inf.
template <typename W2>
__global__ __launch_bounds__(256) void num_recursion_kernel(
    const W2* __restrict__ wi, const int* __restrict__ len,
    const int* __restrict__ ulen, const int* __restrict__ status, int T, int Umax,
    double* __restrict__ a, double* __restrict__ bk, double* __restrict__ Nws,
    float* __restrict__ numerator, int* __restrict__ item_status)
{
    extern __shared__ double sm[];
    const int U1 = Umax + 1;
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool fwd = blockIdx.y == 0;
    const int st = status[b];
    if (st != kItemOk) {
        if (fwd && tid == 0) {
            if (item_status) item_status[b] = st;
            numerator[b] = (st == kItemInfeasible) ? LAST_NEG_INF : __builtin_nanf("");
            Nws[b] = (double)LAST_NEG_INF;
        }
        return;
    }
    if (fwd && tid == 0 && item_status) item_status[b] = kItemOk;
    const int L = len[b], U = ulen[b];
    double* buf0 = sm;
    double* buf1 = sm + U1 + 1;               // one pad cell on the right for bk[u+1]
    const double NI = (double)LAST_NEG_INF;
    const W2* wb = wi + (size_t)b * T * U1;
    if (fwd) {
        double* A = a + (size_t)b * (T + 1) * U1;
        for (int u = tid; u <= U; u += blockDim.x) {
            const double v = u == 0 ? 0.0 : NI;
            buf0[u] = v;
            A[u] = v;
        }
        __syncthreads();
        double* cur = buf0;
        double* nxt = buf1;
        for (int t = 0; t < L; ++t) {
            const W2* wt = wb + (size_t)t * U1;
            for (int u = tid; u <= U; u += blockDim.x) {
                double v = cur[u] + (double)wt[u].x;
                if (u >= 1) v = log_add(v, cur[u - 1] + (double)wt[u - 1].y);
                nxt[u] = v;
                A[(size_t)(t + 1) * U1 + u] = v;
            }
            __syncthreads();
            double* s = cur; cur = nxt; nxt = s;
        }
        if (tid == 0) {
            Nws[b] = cur[U];
            numerator[b] = (float)cur[U];
        }
    } else {
        double* Bk = bk + (size_t)b * (T + 1) * U1;
        for (int u = tid; u <= U + 1; u += blockDim.x) {
            const double v = u == U ? 0.0 : NI;
            buf0[u] = v;
            buf1[u] = NI;
            if (u <= U) Bk[(size_t)L * U1 + u] = v;
        }
        __syncthreads();
        double* cur = buf0;
        double* nxt = buf1;
        for (int t = L - 1; t >= 0; --t) {
            const W2* wt = wb + (size_t)t * U1;
            for (int u = tid; u <= U; u += blockDim.x) {
                const W2 ww = wt[u];
                double v = (double)ww.x + cur[u];
                if (u < U) v = log_add(v, (double)ww.y + cur[u + 1]);
                nxt[u] = v;
                Bk[(size_t)t * U1 + u] = v;
            }
            __syncthreads();
            double* s = cur; cur = nxt; nxt = s;
        }
    }
}

// The same recursion with one wavefront per item and direction, for references of up to
// 64 * CPL - 1 labels: lane l keeps the states u = l*CPL .. l*CPL + CPL-1 of the current frame in
// registers (one lane shuffle per frame hands a value across the lane boundary; no LDS, no
// workgroup barrier), and it reads the gathered arc weights of its states a chunk of CH frames ahead
// of the recursion.  (Pulling them straight out of the dense tensor instead was measured slower:
// every lane then touches two cache lines of its own per frame, and one wavefront cannot keep
// enough of those in flight.)  Arithmetic as in num_recursion_kernel.

template <int CPL, int CH, typename F>
struct NwBuf {
    F w0[CH][CPL], w1[CH][CPL];
};

typedef __amdgpu_buffer_rsrc_t nw_buf_t;
constexpr unsigned kNwOut = 0xfffffff0u;        // a byte offset no buffer of an item reaches: loads give 0, stores are dropped

__device__ __forceinline__ nw_buf_t nw_rsrc(const void* p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(unsigned)bytes, 0x00020000);
}
__device__ __forceinline__ void nw_store64(double v, nw_buf_t r, unsigned voff, unsigned soff)
{
    typedef decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)) b64_t;
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(b64_t, v), r, (int)voff, (int)soff, 0);
}
// log_add without a branch: -inf + -inf stays -inf.  FINE takes the part of the smaller term that 1 + e rounds away
// back in (the locally normalised path, whose gradient is a difference of two such results).
template <bool FINE>
__device__ __forceinline__ double nw_log_add(double x, double y)
{
    const double m = x > y ? x : y;
    const double lo = x > y ? y : x;
    const float d = m == (double)LAST_NEG_INF ? 0.f : (float)(lo - m);
    if (FINE) {
        const float e = __expf(d), u = 1.f + e;
        return m + (double)fmaf(e - (u - 1.f), __builtin_amdgcn_rcpf(u), __logf(u));
    }
    return m + (double)__logf(1.f + __expf(d));
}

// the arc weights of CH frames, t = t0 + k*dir clamped into the item (values of frames outside it are unused)
template <int CPL, int CH, typename F>
__device__ __forceinline__ void nw_load(NwBuf<CPL, CH, F>& d, nw_buf_t irs, unsigned rowb, int t0, int dir, int L,
                                        const unsigned (&ou)[CPL])
{
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        int t = t0 + k * dir;
        t = t < L ? t : L - 1;
        t = t < 0 ? 0 : t;
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            if constexpr (sizeof(F) == 4) {
                const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(irs, (int)ou[i], (int)((unsigned)t * rowb), 0));
                d.w0[k][i] = v.x;
                d.w1[k][i] = v.y;
            } else {
                const double2 v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(irs, (int)ou[i], (int)((unsigned)t * rowb), 0));
                d.w0[k][i] = v.x;
                d.w1[k][i] = v.y;
            }
        }
    }
}

// F = float: gathered weights; double: normalised ones (wi holds pairs of F).
// Requires (T+1)*(Umax+1)*2*sizeof(F) below 2^32 - 16 (byte offsets inside one item's arrays).
template <int CPL, int CH, typename F>
__global__ __launch_bounds__(kWave) void num_wave_kernel(
    const F* __restrict__ wi, const int* __restrict__ len, const int* __restrict__ ulen,
    const int* __restrict__ status, int T, int Umax, double* __restrict__ a, double* __restrict__ bk,
    double* __restrict__ Nws, float* __restrict__ numerator, int* __restrict__ item_status)
{
    const int U1 = Umax + 1;
    const int b = blockIdx.x, lane = threadIdx.x;
    const bool fwd = blockIdx.y == 0;
    const int st = status[b];
    if (st != kItemOk) {
        if (fwd && lane == 0) {
            if (item_status) item_status[b] = st;
            numerator[b] = (st == kItemInfeasible) ? LAST_NEG_INF : __builtin_nanf("");
            Nws[b] = (double)LAST_NEG_INF;
        }
        return;
    }
    if (fwd && lane == 0 && item_status) item_status[b] = kItemOk;
    const int L = len[b], U = ulen[b];
    const double NI = (double)LAST_NEG_INF;
    const unsigned rowb = (unsigned)U1 * 8u, rowi = (unsigned)U1 * (unsigned)(2 * sizeof(F));
    const nw_buf_t irs = nw_rsrc(wi + (size_t)b * T * U1 * 2, (size_t)T * U1 * 2 * sizeof(F));
    // byte offset of each of this lane's states inside a row of the (t,u) arrays and of the weights; kNwOut past the
    // reference
    unsigned ou[CPL], ow[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        const int u = lane * CPL + i;
        ou[i] = u <= U ? (unsigned)u * 8u : kNwOut;
        ow[i] = u <= U ? (unsigned)u * (unsigned)(2 * sizeof(F)) : kNwOut;
    }
    double cur[CPL];
    NwBuf<CPL, CH, F> nxt;
    if (fwd) {
        const nw_buf_t ars = nw_rsrc(a + (size_t)b * (T + 1) * U1, (size_t)(T + 1) * U1 * 8);
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            cur[i] = lane * CPL + i == 0 ? 0.0 : NI;
            nw_store64(cur[i], ars, ou[i], 0);
        }
        if (L > 0) nw_load<CPL, CH, F>(nxt, irs, rowi, 0, 1, L, ow);
        for (int t0 = 0; t0 < L; t0 += CH) {
            const NwBuf<CPL, CH, F> now = nxt;                       // (waits for the chunk, then frees its registers)
            nw_load<CPL, CH, F>(nxt, irs, rowi, t0 + CH, 1, L, ow);
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int t = t0 + k;
                if (t < L) {
                    double up[CPL];
#pragma unroll
                    for (int i = 0; i < CPL; ++i) up[i] = cur[i] + (double)now.w1[k][i];     // label arc u -> u+1
                    double left = __shfl_up(up[CPL - 1], 1, kWave);
                    left = lane == 0 ? NI : left;
#pragma unroll
                    for (int i = 0; i < CPL; ++i) {
                        const double v = nw_log_add<sizeof(F) == 8>(cur[i] + (double)now.w0[k][i], i == 0 ? left : up[i - 1]);
                        cur[i] = v;
                        nw_store64(v, ars, ou[i], (unsigned)(t + 1) * rowb);
                    }
                }
            }
        }
        // N = the forward weight of (L, U)
        double nv = NI;
#pragma unroll
        for (int i = 0; i < CPL; ++i) nv = lane * CPL + i == U ? cur[i] : nv;
        if (lane == U / CPL) {
            Nws[b] = nv;
            numerator[b] = (float)nv;
        }
    } else {
        const nw_buf_t brs = nw_rsrc(bk + (size_t)b * (T + 1) * U1, (size_t)(T + 1) * U1 * 8);
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
            cur[i] = lane * CPL + i == U ? 0.0 : NI;
            nw_store64(cur[i], brs, ou[i], (unsigned)L * rowb);
        }
        // frames walked downwards: the chunk that ends below frame tend holds frames tend-1, tend-2, ...
        if (L > 0) nw_load<CPL, CH, F>(nxt, irs, rowi, L - 1, -1, L, ow);
        for (int tend = L; tend > 0; tend -= CH) {
            const NwBuf<CPL, CH, F> now = nxt;
            nw_load<CPL, CH, F>(nxt, irs, rowi, tend - CH - 1, -1, L, ow);
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int t = tend - 1 - k;
                if (t >= 0) {
                    double right = __shfl_down(cur[0], 1, kWave);
                    right = lane == kWave - 1 ? NI : right;
#pragma unroll
                    for (int i = 0; i < CPL; ++i) {
                        const double nb = i + 1 < CPL ? cur[i + 1] : right;     // still the weight of frame t+1
                        const double v = nw_log_add<sizeof(F) == 8>((double)now.w0[k][i] + cur[i], (double)now.w1[k][i] + nb);
                        cur[i] = v;
                        nw_store64(v, brs, ou[i], (unsigned)t * rowb);
                    }
                }
            }
        }
    }
}

// Marginals of the intersected lattice (Eq. 1 on the (t,u) grid), added with
// the caller's scale onto dw[b][t][ctx(u)][label].  Several u may share one
// arc of the complete lattice, hence atomic adds.
__global__ void num_scatter_kernel(const float2* __restrict__ wi, const int* __restrict__ len,
                                   const int* __restrict__ refs, const int* __restrict__ ulen,
                                   const int* __restrict__ status, const int* __restrict__ ctxs,
                                   Ctx c, int T, int Umax,
                                   const double* __restrict__ a, const double* __restrict__ bk,
                                   const double* __restrict__ Nws, float* __restrict__ dw,
                                   float scale)
{
    const int U1 = Umax + 1;
    const int b = blockIdx.z, t = blockIdx.y;
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= U1 || status[b] != kItemOk) return;
    const int L = len[b], U = ulen[b];
    if (t >= L || u > U) return;
    const double N = Nws[b];
    const double av = a[((size_t)b * (T + 1) + t) * U1 + u];
    if (av == (double)LAST_NEG_INF || N == (double)LAST_NEG_INF) return;
    const int* r = refs + (size_t)b * Umax;
    const int q = ctxs[(size_t)b * U1 + u];
    const float2 ww = wi[((size_t)b * T + t) * U1 + u];
    float* row = dw + (((size_t)b * T + t) * c.C + q) * c.V1;
    const double* bn = bk + ((size_t)b * (T + 1) + t + 1) * U1;
    const double e0 = av + (double)ww.x + bn[u] - N;
    if (e0 > -100.0) atomicAdd(row, scale * __expf((float)e0));
    if (u < U) {
        const double e1 = av + (double)ww.y + bn[u + 1] - N;
        if (e1 > -100.0) atomicAdd(row + r[u], scale * __expf((float)e1));
    }
}

// Gradient of the locally normalised log-likelihood (Section 2.1) with respect to the weights,
// dw[b][t][q][y] (+)= scale * ( [marginals of the intersected lattice riding on arc (t,q,y)]
//                              - [their sum over the arcs leaving (t,q)] * softmax(w[b][t][q])[y] ).
// One workgroup per frame, several where the frames are large and few (each forms the marginals of all cells and takes
// its share of the rows: one item, 10 frames, 2001 labels 247 -> 47 us, 50 frames of 1201 labels 161 -> 71 us): the
// marginals of its cells first (thread <-> cell, into LDS), then row by row one
// wavefront per chain of cells with the same context q (see num_check_kernel): it alone writes row (t,q), so no
// atomics are needed and the result does not depend on timing.  Rows that no path visits are zero (accumulate:
// left alone) and are written by the same workgroup, every element of the tensor once.
// Bound: HBM, the tensor written once and the visited rows read.  B=16, T=500, V=256, 50 to 150 labels: 1.19 -> 0.69 ms
// against a fill of the whole tensor followed by a wavefront per chain whose cells were fetched one by one.  ORDERED: rows are
// written in their order, zeros or not (0.705 -> 0.66 ms against the zeros of a frame first): what a frame's zeros leave out costs as much as what they write.  (The
// zero rows alone, beside the recursion: 1.4 GB in 0.43 ms, while the whole 2.1 GB go in 0.33.)
// zeroed: the tensor has been filled with zeros by another kernel (context sets too large for `seen`).
// LDS: float2[U1] marginals | int[U1] links | int[U1] labels | ORDERED: short[C] head of the row's chain, -1: not visited; else
// int[U1] heads of visited chains | unsigned char[C] visited (unless zeroed or accumulated).
constexpr int kNsThreads = 512;
constexpr int kNsMaxC = 32768;
template <int QL, bool ORDERED>
__global__ __launch_bounds__(kNsThreads) void num_scatter_local_kernel(
    const float* __restrict__ w, const double2* __restrict__ wd, const double* __restrict__ lz,
    const int* __restrict__ len, const int* __restrict__ refs, const int* __restrict__ ulen,
    const int* __restrict__ status, const int* __restrict__ ctxs, const int* __restrict__ link,
    Ctx c, int T, int Umax, const double* __restrict__ a, const double* __restrict__ bk,
    const double* __restrict__ Nws, float* __restrict__ dw, float scale, int accumulate, int zeroed)
{
    extern __shared__ float2 nsl_p[];
    __shared__ int count, visited;
    const int U1 = Umax + 1;
    int* next = (int*)(nsl_p + U1);             // next cell of the chain, -1: none
    int* label = next + U1;                     // label of the cell's label arc, -1: none
    short* head = (short*)(label + U1);
    int* heads = label + U1;
    unsigned char* seen = (unsigned char*)(heads + U1);
    const bool zeros = !accumulate && !zeroed;  // rows no path visits are written here
    const int b = blockIdx.y, t = blockIdx.x, tid = threadIdx.x, part = blockIdx.z, parts = gridDim.z;
    const int wv = tid / kWave, lane = tid & (kWave - 1);
    constexpr int NW = kNsThreads / kWave;
    const int L = len[b], U = ulen[b];
    const double N = status[b] == kItemOk ? Nws[b] : (double)LAST_NEG_INF;
    const bool live = N != (double)LAST_NEG_INF && t < L;
    if (!live && !zeros) return;
    const size_t fo = ((size_t)b * T + t) * c.C * c.V1;
    const int* r = refs + (size_t)b * Umax;
    const int* lk = link + (size_t)b * U1 * 2;
    const int* cx = ctxs + (size_t)b * U1;
    const size_t cell0 = ((size_t)b * T + t) * U1;
    if constexpr (ORDERED) {
        for (int q = tid; q < c.C; q += kNsThreads) head[q] = -1;
    } else if (zeros) {
        for (int q = tid; q < c.C; q += kNsThreads) seen[q] = 0;
    }
    if (tid == 0) { count = 0; visited = 0; }
    if (live) {
        const double* at = a + ((size_t)b * (T + 1) + t) * U1;
        const double* bn = bk + ((size_t)b * (T + 1) + t + 1) * U1;
        for (int v = tid; v <= U; v += kNsThreads) {
            const double av = at[v];
            float2 p = make_float2(0.f, 0.f);
            if (av != (double)LAST_NEG_INF) {
                const double2 ww = wd[cell0 + v];
                const double e0 = av + ww.x + bn[v] - N;
                if (e0 > -100.0) p.x = __expf((float)e0);
                if (v < U) {
                    const double e1 = av + ww.y + bn[v + 1] - N;
                    if (e1 > -100.0) p.y = __expf((float)e1);
                }
            }
            // a cell that no path reaches, or outside the cone of paths (it carries no log-sum-exp): not visited
            if (av == (double)LAST_NEG_INF || v > t || U - v > L - t) p.x = -1.f;
            nsl_p[v] = p;
            next[v] = lk[2 * v];
            label[v] = v < U ? r[v] : -1;
        }
    }
    __syncthreads();
    if (live)
        for (int u = tid; u <= U; u += kNsThreads) {
            if (!lk[2 * u + 1]) continue;
            bool any = false;
            for (int v = u; v >= 0 && !any; v = next[v]) any = nsl_p[v].x >= 0.f;
            if (!any) continue;
            visited = 1;
            if constexpr (ORDERED) {
                head[cx[u]] = (short)u;                                 // (fewer than 4096 labels)
                continue;
            }
            if (u % parts == part) heads[atomicAdd(&count, 1)] = u;     // (the order of the rows does not matter)
            if (zeros) seen[cx[u]] = 1;
        }
    __syncthreads();
    const int n = live ? count : 0;
    // rows no path visits
    if (zeros) {
        float* g = dw + fo;
        if (!live || !visited) {
            const int total = c.C * c.V1, lead = min((int)((4 - ((size_t)g >> 2)) & 3), total), n4 = (total - lead) / 4;
            for (size_t i = (size_t)part * kNsThreads + tid; i < (size_t)n4; i += (size_t)parts * kNsThreads)
                *(float4*)(g + lead + 4 * i) = make_float4(0.f, 0.f, 0.f, 0.f);
            if (part > 0) return;
            if (tid < lead) g[tid] = 0.f;
            for (int i = lead + 4 * n4 + tid; i < total; i += kNsThreads) g[i] = 0.f;
            return;
        }
    }
    auto zero_row = [&](float* grow) __attribute__((always_inline)) {
        struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
        for (int y = 4 * lane; y < c.V1; y += 4 * kWave)
            if (c.V1 >= 4) *(f4*)(grow + min(y, c.V1 - 4)) = f4{{0.f, 0.f, 0.f, 0.f}};
            else
                for (int k = y; k < c.V1; ++k) grow[k] = 0.f;
    };
    constexpr int Q = QL > 0 ? QL : 2;
    const NumPieces<Q> p(c.V1, lane);
    auto row = [&](int u, size_t ro, const NumRow<Q>& x) __attribute__((always_inline)) {
        float occ = 0.f, pbs = 0.f, lab[Q][4];
        int first = -1;
        // the chain's label marginals by column, in chain order (deterministic), and once per row their sums
        auto walk = [&](const NumPieces<Q>& at, bool sums) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) lab[j][k] = 0.f;
            for (int v = u; v >= 0; v = next[v]) {
                const float2 pv = nsl_p[v];
                const int y = label[v];
                if (pv.x < 0.f) continue;
                if (sums) {
                    if (first < 0) first = v;
                    occ += pv.x + pv.y;
                    pbs += pv.x;
                }
#pragma unroll
                for (int j = 0; j < Q; ++j)
#pragma unroll
                    for (int k = 0; k < 4; ++k) lab[j][k] += at.at[j] + k == y ? pv.y : 0.f;
            }
        };
        walk(p, true);
        const double z = lz[cell0 + first];                    // the same for every cell of the chain
        float* grow = dw + ro;
        auto grad = [&](int y, float wy, float l) __attribute__((always_inline)) {
            const float g = l - occ * __expf((float)((double)wy - z));
            return scale * (y == 0 ? g + pbs : g);
        };
        auto put = [&](const NumPieces<Q>& at, const NumRow<Q>& r) __attribute__((always_inline)) {
            struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                if (at.skip[j] >= 4) continue;
                f4 o;
#pragma unroll
                for (int k = 0; k < 4; ++k) o.v[k] = grad(at.at[j] + k, r.w[j][k], lab[j][k]);
                float* d = grow + at.at[j];
                if (!accumulate) *(f4*)d = o;
                else
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (k >= at.skip[j]) d[k] += o.v[k];
            }
        };
        if (QL > 0) {
            put(p, x);
        } else if (c.V1 >= 4) {
            // (one walk along the chain per stretch: with one per 64 columns 4000 labels took 3 times as long)
            for (int c0 = 0; c0 < c.V1; c0 += 4 * kWave * Q) {
                const NumPieces<Q> at(c.V1, lane, c0);
                const NumRow<Q> r = num_load_row<Q>(w + ro, at);
                if (c0 > 0) walk(at, false);
                put(at, r);
            }
        } else {
            for (int y = lane; y < c.V1; y += kWave) {
                float l = 0.f;
                for (int v = u; v >= 0; v = next[v])
                    if (nsl_p[v].x >= 0.f && label[v] == y) l += nsl_p[v].y;
                const float o = grad(y, w[ro + y], l);
                if (accumulate) grow[y] += o; else grow[y] = o;
            }
        }
    };
    if constexpr (!ORDERED) {
        if (zeros)
            for (int q = part * NW + wv; q < c.C; q += parts * NW)
                if (!seen[q]) zero_row(dw + fo + (size_t)q * c.V1);
        auto row_of = [&](int i) __attribute__((always_inline)) { return fo + (size_t)cx[heads[min(i, n - 1)]] * c.V1; };
        NumRow<Q> nx;
        if (QL > 0 && n > 0) nx = num_load_row<Q>(w + row_of(wv), p);
        for (int i = wv; i < n; i += NW) {
            const NumRow<Q> x = nx;
            if (QL > 0) nx = num_load_row<Q>(w + row_of(i + NW), p);
            row(heads[i], row_of(i), x);
        }
    } else {
        // own rows first + step i; those of the next 64 that are visited as a mask, the weights of the next one requested while one
        // is worked on
        const int first = part * NW + wv, step = parts * NW;
        for (int q0 = first; q0 < c.C; q0 += step * kWave) {
            const int mine = q0 + step * lane, h = mine < c.C ? head[mine] : -1;
            unsigned long long m = __ballot(h >= 0);
            const int rows = min(kWave, (c.C - q0 + step - 1) / step);
            NumRow<Q> nx;
            auto request = [&](int i) __attribute__((always_inline)) {
                if (QL > 0) nx = num_load_row<Q>(w + fo + (size_t)(q0 + step * i) * c.V1, p);
            };
            int at = m ? __ffsll(m) - 1 : kWave;
            if (at < kWave) request(at);
            for (int i = zeros ? 0 : at; i < rows; zeros ? ++i : i = at) {
                const size_t ro = fo + (size_t)(q0 + step * i) * c.V1;
                if (i == at) {
                    const NumRow<Q> x = nx;
                    m &= m - 1;
                    at = m ? __ffsll(m) - 1 : kWave;
                    request(min(at, rows - 1));
                    row(__builtin_amdgcn_readlane(h, i), ro, x);
                    continue;
                }
                zero_row(dw + ro);
            }
        }
    }
}

}  // namespace last
