// On-the-fly weights of the shared-embedding function for whole stretches of frames, laid out in memory
//     w[t][q][y] = sum_k bf16(tanh(f[t][k] + e[q][k])) W[k][y]
// for the recursions of trigram_kernels.hpp, and the gradients of f, e and W from the vectors that those leave.
//
// The kernels of fused_kernels.hpp form the hidden vectors inside the chain of the recursion, three times, and send
// them through LDS.  Here nothing but the recursion (2.0 us a frame) is serial: the hidden units, of which there are H / (V+1)
// for every arc, are formed at the rate of the vector ALU by the whole chip, in the registers of the lane that feeds them to
// the matrix cores, once for the weights and once for the gradients.  4 bytes an arc are written once and read three times
// (by both directions and for the gradients; once for a distance, whose directions meet in the middle): 1.35 of 11.0 ms.
// 16 items, 1024 frames, 32 labels, 512 hidden units: loss with gradients 42.3 -> 11.0 ms (weights 1.75, recursions 2.0,
// gradients 6.9); distance of 4 items, 1000 frames, 64 labels 7.4 -> 3.94 ms (weights 2.4, recursions 1.6).
//
// In the weights tanh(f + e) = 1 - 2 / (1 + e^2f e^2e), with e^2f and e^2e formed once per element of f and e, is a product
// and a sum in one instruction, one reciprocal and one more instruction.  Both factors are held within e^+-80: where |f| or
// |e| is above 40 and the other is below 30 the sum saturates just the same; where both f and e have values above 30 (no such
// sum need saturate) the exponential of each sum is taken (`wide`).
#include <algorithm>
#include <mutex>
#include <set>
#include <utility>

#include "common.hpp"
#include "emb.hpp"

namespace last {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr float kTwoLog2e = 2.885390081777926814f;
constexpr float kEmClamp = 40.f;     // e^80 and e^-80 are float32 values
constexpr float kEmLarge = 30.f;
constexpr int kEwWaves = 8;          // weights kernel: waves of a workgroup
// frames of a wave at a time: the accumulators of 8 (6) row tiles by NT label tiles are 32 to 128 registers
template <int NT> constexpr int kEwFrames = NT < 5 ? 4 : 3;

__device__ __forceinline__ float bf_lo(unsigned pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf_hi(unsigned pair) { return __uint_as_float(pair & 0xffff0000u); }

inline __host__ __device__ int label_tiles(int V) { return (V + 1 + 15) / 16; }
// steps of 16 labels of the gradient kernel's contraction over the labels (two instantiations)
inline __host__ __device__ int grad_steps(int V) { return V <= 32 ? 2 : 4; }

// the same from the sum f + e
__device__ __forceinline__ float em_tanh(float x)
{
    return fmaf(-2.f, __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x * kTwoLog2e)), 1.f);
}

// WIDE: f, e are the values themselves, otherwise their exponentials e^2f, e^2e
template <bool WIDE>
__device__ __forceinline__ float em_tanh(float f, float e)
{
    if (WIDE) return em_tanh(f + e);
    const float d = fmaf(f, e, 1.f);
    return fmaf(-2.f, __builtin_amdgcn_rcpf(d), 1.f);
}

// What the other kernels start from, in one launch (a call of a few frames is launches for the most part):
//   e^2f, e^2e, and whether f (of the frames that exist: what lies behind an item's end has no part in the results) and e
//   have large values;
//   W repacked as operand fragments, lane l of (ks, nt):
//     Wn[ks][nt][l] = W[32 ks + 8 (l / 16) + j][16 nt + l % 16],
//     Wt[ht][ky][l] = W[32 ht + l % 32][16 ky + 8 (l / 32) + j + 1],       j = 0..7, zero outside W;
//   the list of the frames that exist (item by item);
//   the cleared exchange area and flags of the recursions.
__global__ __launch_bounds__(256) void emb_prepare_kernel(EmbArgs a, size_t nf, size_t ne, size_t ne_pad, int NT)
{
    __shared__ int s_or[4];
    __shared__ int s_sum[4];
    const int tid = threadIdx.x;
    for (size_t i = (size_t)blockIdx.x * 256 + tid; i < a.xwords; i += (size_t)kEmScan * 256) a.x[i] = ~0ull;
    for (int i = blockIdx.x * 256 + tid; i < a.B; i += kEmScan * 256) a.fail[i] = 0;
    auto value = [&](float x) __attribute__((always_inline)) {
        const float c = fminf(fmaxf(x, -kEmClamp), kEmClamp);
        // (rounded once: with the exponential of a rounded product the tanh of large f and e was off by 6e-7)
        return x != x ? x : (float)exp(2.0 * (double)c);
    };
    auto fill = [&](const unsigned* src, float* dst, size_t n, size_t n_pad, auto&& counts) {
        bool big = false;
#pragma unroll 2
        for (size_t i = (size_t)blockIdx.x * 256 + tid; i < n_pad / 8; i += (size_t)kEmScan * 256) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (8 * i < n) v = ((const u32x4*)src)[i];
            bool l = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) l = l | (fabsf(bf_lo(v[j])) > kEmLarge) | (fabsf(bf_hi(v[j])) > kEmLarge);
            big = big | (l & counts((unsigned)i));           // (fewer than 2^32 pieces: 8 GiB hold the weights of their frames)
            float4* d = (float4*)(dst + 8 * i);
            d[0] = make_float4(value(bf_lo(v[0])), value(bf_hi(v[0])), value(bf_lo(v[1])), value(bf_hi(v[1])));
            d[1] = make_float4(value(bf_lo(v[2])), value(bf_hi(v[2])), value(bf_lo(v[3])), value(bf_hi(v[3])));
        }
        return big;
    };
    auto frame_exists = [&](unsigned i) {
        const unsigned row = i / (unsigned)(a.H / 8), b = row / (unsigned)a.T;
        const int L = a.len[b];
        return L <= a.T && (int)(row - b * (unsigned)a.T) < L;
    };
    const bool le = fill((const unsigned*)a.e, a.Ee, ne, ne_pad, [](unsigned) { return true; });
    const bool lf = fill((const unsigned*)a.f, a.Ef, nf, nf, frame_exists);
    const int any = (__any(lf) ? 1 : 0) | (__any(le) ? 2 : 0);
    if ((tid & 63) == 0) s_or[tid >> 6] = any;
    const __bf16* W = (const __bf16*)a.W;
    const int V1 = a.V + 1, npack = (a.H / 32) * NT * 64;
    for (int i = blockIdx.x * 256 + tid; i < npack; i += kEmScan * 256) {
        const int lane = i & 63, nt = (i >> 6) % NT, ks = (i >> 6) / NT;
        const int y = 16 * nt + (lane & 15);
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 32 * ks + 8 * (lane >> 4) + j;
            v[j] = y < V1 ? W[(size_t)k * V1 + y] : (__bf16)0.f;
        }
        ((bf16x8*)a.Wn)[i] = v;
    }
    const int KY = grad_steps(a.V), npackt = a.Wt ? (a.H / 32) * KY * 64 : 0;
    for (int i = blockIdx.x * 256 + tid; i < npackt; i += kEmScan * 256) {
        const int lane = i & 63, ky = (i >> 6) % KY, ht = (i >> 6) / KY;
        const int k = 32 * ht + (lane & 31);
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int y = 16 * ky + 8 * (lane >> 5) + j + 1;
            v[j] = y < V1 ? W[(size_t)k * V1 + y] : (__bf16)0.f;
        }
        ((bf16x8*)a.Wt)[i] = v;
    }
    for (int b = blockIdx.x; b < a.B; b += kEmScan) {
        int before = 0;
        for (int i = tid; i < b; i += 256) before += a.len[i] < 0 || a.len[i] > a.T ? 0 : a.len[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        __syncthreads();
        if ((tid & 63) == 0) s_sum[tid >> 6] = before;
        __syncthreads();
        const int first = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        const int Lb = a.len[b], n = Lb < 0 || Lb > a.T ? 0 : Lb;
        for (int t = tid; t < n; t += 256) a.frames[first + t] = make_int2(b * a.T + t, b);
        if (b == a.B - 1 && tid == 0) a.count[0] = first + n;
    }
    __syncthreads();
    if (tid == 0) a.big[blockIdx.x] = s_or[0] | s_or[1] | s_or[2] | s_or[3];
}

typedef __amdgpu_buffer_rsrc_t em_buf;

__device__ __forceinline__ em_buf em_make_buf(const void* p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float em_load(em_buf r, unsigned off)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ void em_store(float x, em_buf r, unsigned voff, unsigned soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, x), r, (int)voff, (int)soff, 0);
}

// One workgroup: 32 states and a stretch of the frame list.  The rows of e^2e (64 KiB) and W (48 to 80 KiB) sit in LDS
// in operand order; a wave takes four frames (three with five label tiles) at a time, so that each fragment of W serves
// eight row tiles of 16, and never meets the others.  A operand: lane l holds hidden units 8 (l / 16) .. + 7 of a step
// of 32 for state l % 16.
// Bound: vector ALU (per hidden unit two fused instructions, a reciprocal of twice a plain instruction's time, half a
// conversion: 1.2 of the 1.9 ms at 16 items, 1024 frames, 32 labels; matrix cores 0.35).  f is requested a step ahead, also
// across groups of frames (2.04 -> 1.89 ms; with five label tiles 2.56 -> 2.32).  LDS operands a step ahead gained nothing.
template <int NT, bool WIDE>
__device__ __forceinline__ void emb_weights_body(const EmbArgs& a, const f32x4* Es, const bf16x8* Ws, int tile, int lo, int hi)
{
    constexpr int FR = kEwFrames<NT>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int H = a.H, V1 = a.V + 1, KS = H / 32;
    const int q0 = tile * kEmTile;
    const size_t fr = (size_t)a.C * V1;
    const int y = lane & 15;
    const unsigned wOff = 4u * (unsigned)(4 * (lane >> 4) * V1 + y), wLast = 16 * (NT - 1) + y < V1 ? wOff : 0x80000000u;
    // frames of the group that starts at list entry i (past the end: the last frame again)
    auto rows_at = [&](int i, int (&row)[FR]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < FR; ++j) row[j] = a.frames[min(i + j, hi - 1)].x;
    };
    const unsigned foff = 8u * (lane >> 4);
    auto request = [&](f32x4 (&x)[2], int row, int k) __attribute__((always_inline)) {
        if (WIDE) {
            const u32x4 v = *(const u32x4*)((const unsigned short*)a.f + (size_t)row * H + k + foff);
            x[0] = f32x4{bf_lo(v[0]), bf_hi(v[0]), bf_lo(v[1]), bf_hi(v[1])};
            x[1] = f32x4{bf_lo(v[2]), bf_hi(v[2]), bf_lo(v[3]), bf_hi(v[3])};
            return;
        }
        const float* p = a.Ef + (size_t)row * H + k;
        x[0] = *(const f32x4*)(p + foff);
        x[1] = *(const f32x4*)(p + foff + 4);
    };
    const int first = lo + FR * wave;
    if (first >= hi) return;
    int row[FR], next[FR];
    f32x4 nx[FR][2];
    rows_at(first, next);
#pragma unroll
    for (int j = 0; j < FR; ++j) {
        next[j] = __builtin_amdgcn_readfirstlane(next[j]);
        request(nx[j], next[j], 0);
    }
    for (int i = first; i < hi; i += FR * kEwWaves) {
        int after[FR];
        rows_at(i + FR * kEwWaves, after);
#pragma unroll
        for (int j = 0; j < FR; ++j) row[j] = next[j];
        f32x4 acc[2][FR][NT];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < FR; ++j)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[h][j][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks) {
            // f of the next step, and in the last one of the next group's first step, is requested a step ahead
            const bool last = ks + 1 == KS;
            if (ks == 0) {
#pragma unroll
                for (int j = 0; j < FR; ++j) next[j] = __builtin_amdgcn_readfirstlane(after[j]);
            }
            f32x4 ee[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 2; ++g) ee[h][g] = Es[((ks * 2 + h) * 2 + g) * 64 + lane];
            bf16x8 wf[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) wf[n] = Ws[(ks * NT + n) * 64 + lane];
#pragma unroll
            for (int j = 0; j < FR; ++j) {
                const f32x4 x[2] = {nx[j][0], nx[j][1]};
                request(nx[j], last ? next[j] : row[j], last ? 0 : 32 * (ks + 1));
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4 hv;
#pragma unroll
                    for (int g = 0; g < 2; ++g)
#pragma unroll
                        for (int c = 0; c < 4; c += 2) {
                            const f32x2 p = {em_tanh<WIDE>(x[g][c], ee[h][g][c]), em_tanh<WIDE>(x[g][c + 1], ee[h][g][c + 1])};
                            hv[2 * g + c / 2] = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2));
                        }
                    const bf16x8 av = __builtin_bit_cast(bf16x8, hv);
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[h][j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, wf[n], acc[h][j][n], 0, 0, 0);
                }
                if (NT > 3) __builtin_amdgcn_sched_barrier(0);            // (registers)
            }
        }
        // states past the last one are past the end of the descriptor (checked with the uniform part of the offset), labels
        // past the last one get an offset that is so anywhere
#pragma unroll
        for (int j = 0; j < FR; ++j) {
            const em_buf o = em_make_buf(a.w + (size_t)row[j] * fr + (size_t)q0 * V1, i + j < hi ? 4u * (unsigned)((a.C - q0) * V1) : 0u);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        em_store(acc[h][j][n][r], o, (n < NT - 1 ? wOff : wLast) + 64u * n, 4u * (unsigned)((16 * h + r) * V1));
        }
    }
}

template <int NT>
__global__ __launch_bounds__(64 * kEwWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void emb_weights_kernel(EmbArgs a)
{
    extern __shared__ __align__(16) unsigned char em_smem[];
    const int H = a.H, KS = H / 32;
    f32x4* Es = (f32x4*)em_smem;                   // [KS][2][2][64]
    bf16x8* Ws = (bf16x8*)(Es + KS * 256);         // [KS][NT][64]
    const int tile = blockIdx.x % a.tiles, ch = blockIdx.x / a.tiles;
    const long long n = a.count[0];
    const int lo = (int)(n * ch / a.nch), hi = (int)(n * (ch + 1) / a.nch);
    if (lo >= hi) return;
    static_assert(kEmScan == 2 * 64 * kEwWaves, "two words a thread");
    const int large = a.big[threadIdx.x] | a.big[threadIdx.x + 64 * kEwWaves];
    for (int i = threadIdx.x; i < KS * 256; i += 64 * kEwWaves) {
        const int l = i & 63, g = (i >> 6) & 1, h = (i >> 7) & 1, ks = i >> 8;
        Es[i] = *(const f32x4*)(a.Ee + (size_t)(tile * kEmTile + 16 * h + (l & 15)) * H + 32 * ks + 8 * (l >> 4) + 4 * g);
    }
    for (int i = threadIdx.x; i < KS * NT * 64; i += 64 * kEwWaves) Ws[i] = ((const bf16x8*)a.Wn)[i];
    const int in_f = __syncthreads_or(large & 1), in_e = __syncthreads_or(large & 2);
    if (!in_f || !in_e) {
        emb_weights_body<NT, false>(a, Es, Ws, tile, lo, hi);
        return;
    }
    // both f and e have large values: e itself in the place of its exponentials
    for (int i = threadIdx.x; i < KS * 256; i += 64 * kEwWaves) {
        const int l = i & 63, g = (i >> 6) & 1, h = (i >> 7) & 1, ks = i >> 8, q = tile * kEmTile + 16 * h + (l & 15);
        const unsigned* p = (const unsigned*)a.e + ((size_t)min(q, a.C - 1) * H + 32 * ks + 8 * (l >> 4) + 4 * g) / 2;
        Es[i] = f32x4{bf_lo(p[0]), bf_hi(p[0]), bf_lo(p[1]), bf_hi(p[1])};
    }
    __syncthreads();
    emb_weights_body<NT, true>(a, Es, Ws, tile, lo, hi);
}

// ---- the gradient ---------------------------------------------------------------------------------

typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ float em_exp(float x) { return __builtin_amdgcn_exp2f(x * (0.5f * kTwoLog2e)); }
__device__ __forceinline__ void em_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// partition sum of every frame from the two vectors at hand (see dense_marginals_kernel); one wavefront a frame
__global__ __launch_bounds__(256) void emb_norm_kernel(EmbArgs a, EmbGradArgs g)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= a.count[0]) return;
    const int2 fr = a.frames[i];
    const size_t ra = (size_t)fr.x + fr.y;                        // row b (T + 1) + t
    const float* al = g.alpha + (ra + 1) * a.C;
    const float* be = g.beta + (ra + 1) * a.C;
    float m = LAST_NEG_INF, z = 0.f;
    for (int q = lane; q < a.C; q += 64) {
        const float a1 = al[q], v = a1 == LAST_NEG_INF ? a1 : a1 + be[q];
        const float n = fmaxf(m, v), nn = n == LAST_NEG_INF ? 0.f : n;
        z = fmaf(z, em_exp(m - nn), em_exp(v - nn));
        m = n;
    }
    const float M = wave_max(m), MM = M == LAST_NEG_INF ? 0.f : M;      // (no path: every exponential below is zero)
    z = wave_sum(z * em_exp(m - MM));
    if (lane == 0) {
        EmbNorm n;
        n.k = g.offa[ra] - g.offa[ra + 1] - (double)MM;
        n.iz = M == LAST_NEG_INF ? 1.f : 1.f / z;
        n.unused = 0.f;
        g.norm[fr.x] = n;
    }
}

// marginals of the two arcs that leave every cell (t, u) of the intersected lattice, in the place of their weights
__global__ __launch_bounds__(256) void emb_cell_marginals_kernel(EmbArgs a, EmbNumArgs n, int t0)
{
    const int U1 = n.U1, b = blockIdx.z, t = t0 + blockIdx.y;
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= U1 || n.status[b] != kItemOk) return;
    const int L = a.len[b], U = n.ulen[b];
    if (t >= L || u > U) return;
    const size_t cell = ((size_t)b * a.T + t) * U1 + u;
    const double N = n.N[b], av = n.a[((size_t)b * (a.T + 1) + t) * U1 + u];
    float2 p = make_float2(0.f, 0.f);
    if (av != (double)LAST_NEG_INF && N != (double)LAST_NEG_INF) {
        const float2 ww = n.wi[cell];
        const double* bn = n.bk + ((size_t)b * (a.T + 1) + t + 1) * U1;
        const double e0 = av + (double)ww.x + bn[u] - N;
        if (e0 > -100.0) p.x = __expf((float)e0);
        if (u < U) {
            const double e1 = av + (double)ww.y + bn[u + 1] - N;
            if (e1 > -100.0) p.y = __expf((float)e1);
        }
    }
    n.wi[cell] = p;
}

// cells of every item by the tile of their state; LDS: int[tiles + 1]
__global__ __launch_bounds__(256) void emb_cells_kernel(EmbArgs a, EmbNumArgs n)
{
    extern __shared__ int em_cnt[];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int cells = n.status[b] == kItemOk ? n.ulen[b] + 1 : 0;
    int* st = n.starts + (size_t)b * (a.tiles + 1);
    for (int i = tid; i <= a.tiles; i += 256) em_cnt[i] = 0;
    __syncthreads();
    for (int u = tid; u < cells; u += 256) atomicAdd(em_cnt + n.ctxs[(size_t)b * n.U1 + u] / kEmTile, 1);
    __syncthreads();
    if (tid == 0) {
        int sum = 0;
        for (int i = 0; i <= a.tiles; ++i) {
            const int c = em_cnt[i];
            em_cnt[i] = sum;
            st[i] = sum;
            sum += c;
        }
    }
    __syncthreads();
    for (int u = tid; u < cells; u += 256) {
        const int q = n.ctxs[(size_t)b * n.U1 + u];
        const int y = u + 1 < cells ? n.refs[(size_t)b * (n.U1 - 1) + u] : 0;
        n.cells[(size_t)b * n.U1 + atomicAdd(em_cnt + q / kEmTile, 1)] = u << 12 | (q % kEmTile) << 7 | y;
    }
}

// Chain of the arc marginals through the weight function.  With h = bf16(tanh(f_t + e_q)) and g the marginals (minus
// those of the intersected lattice),
//   dW[k][y] += h[k] g[q][y],   d[q][k] = (sum_y g[q][y] W[k][y]) (1 - h[k]^2),   de[q] += d[q],   df[t] += sum_q d[q]
// (the rounding of h is the identity when differentiating).  g enters the matrix cores as two bf16 parts, 16 bits, and as three,
// all 24, where an intersected lattice is subtracted: its marginals are near 1 on a few arcs, so that 16 bits of them showed
// (error of df five times that of float32 arithmetic).
// One workgroup: 32 states, all hidden units (64 a wave), a stretch of the frame list.  d comes out of the matrix cores
// with lane l holding hidden unit l % 32 for 16 of the 32 states; h is formed for just these, so e and de stay in
// registers for all frames, f is one value a lane, and the same registers, read as an operand whose contraction runs
// over states in that order, form dW.  The hidden tile never goes through LDS; the marginals do, formed by
// the workgroup one frame ahead from the weights and the two state vectors and stored in the two operand orders.
// The empty label, which would open another tile of 16 or 32 labels, goes through the vector ALU.
// The hidden units are rounded here exactly as the numerator's kernels round theirs (em_tanh of the sum, two
// transcendental instructions): 1 - h^2 of a unit that rounds the other way is off by up to 2^-7, and where one state holds
// most of a frame's weight that is 1.6e-3 of an element of df.  (In the weights the same unit moves a sum of H
// by 2^-9 W: there the product of exponentials does.  Of units above 2^-8, sigma 1 and 0.5, 2.7e-6 round the other way than in 64
// bits, 2.9e-6 with the exponential of the sum; of the smaller ones 5e-5 and 2e-6.)
// Sums over states and over frames leave as partial sums for emb_sum_kernel.
// Bound (without the third part): vector ALU, 13 instructions and two transcendental ones a hidden unit, 4.0 of 6.1 ms at 16 items, 1024 frames, 32 labels,
// 512 hidden units (matrix cores 0.9); two waves a SIMD (256 registers) leave the rest as waits for LDS.  Every load is issued on
// every path, so that the waits are counted (with a condition around the cells' loads 6.9 ms); all LDS reads of a frame ahead
// of the hidden units spilled (6.3 to 6.9).  Two frames between barriers up to 32 labels 6.2 -> 6.1.  In a loss the third part
// and de put away with dW cost 8 % of the call (10.85 -> 11.75 ms; 4x400 frames, 64 labels 6.6 -> 7.2); operands of the third
// part read where they are used, or the small parts first, 11.85 to 11.95.
template <int NW, int KY, bool NUM>
struct EmGradLds {
    static constexpr int P = NUM ? 3 : 2;          // bf16 parts of a marginal
    static constexpr int S1 = 16 * KY + 8;         // row strides (bf16): 16-byte reads of 8 lanes fall on different banks
    static constexpr int S2 = 40;
    static constexpr int NT = KY / 2;              // tiles of 32 labels
    static constexpr int FP = KY == 2 ? 2 : 1;     // frames between two barriers
    __bf16 g1[2 * FP][P][32 * S1];                 // [buffer][part][state][label - 1]
    __bf16 g2[2 * FP][P][32 * NT * S2];            // [buffer][part][label - 1][state in operand order]
    float g0[2 * FP][32];                          // empty label
    float num[NUM ? 2 * FP : 1][32 * (16 * KY + 1)];   // marginals of the intersected lattice [state][label]
};

template <int NW, int KY, bool NUM>
__device__ __forceinline__ void emb_grad_body(const EmbArgs& a, const EmbGradArgs& g, EmGradLds<NW, KY, NUM>& s, int tile, int grp, int lo, int hi)
{
    typedef EmGradLds<NW, KY, NUM> S;
    constexpr int NT = S::NT, S1 = S::S1, S2 = S::S2, FP = S::FP, P = S::P;
    constexpr int LPR = 2 * NW;                             // lanes of a row when the marginals are formed
    constexpr int NS = (16 * KY + 1 + LPR - 1) / LPR;       // labels of such a lane
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int V = a.V, V1 = V + 1, C = a.C, H = a.H;
    const int q0 = tile * kEmTile;
    const int k0 = 64 * wave + (lane & 31);
    const size_t fr = (size_t)C * V1;

    // hidden units k0, k0 + 32
    // (with two tiles of labels e stays in pairs of bfloat16: 16 registers less, 32 instructions a frame more)
    constexpr bool PAIRS = KY > 2;
    float ee[PAIRS ? 1 : 2][PAIRS ? 1 : 16], w0[2];
    unsigned ep[PAIRS ? 2 : 1][PAIRS ? 8 : 1];
    bf16x8 wt[2][KY];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const unsigned v = ((const unsigned short*)a.e)[(size_t)min(q0 + (r & 3) + 8 * (r >> 2) + 4 * half, C - 1) * H + k0 + 32 * kt];
            if constexpr (!PAIRS) ee[kt][r] = bf_lo(v);
            else ep[kt][r >> 1] = r & 1 ? ep[kt][r >> 1] | v << 16 : v;
        }
#pragma unroll
        for (int ky = 0; ky < KY; ++ky) wt[kt][ky] = ((const bf16x8*)a.Wt)[((2 * wave + kt) * KY + ky) * 64 + lane];
        w0[kt] = (float)((const __bf16*)a.W)[(size_t)(k0 + 32 * kt) * V1];
    }
    f32x16 de[2], dw[2][NT];
    float dw0[2] = {0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
        de[kt] = f32x16{};
#pragma unroll
        for (int n = 0; n < NT; ++n) dw[kt][n] = f32x16{};
    }
    // the row of the marginals that this thread forms, and its labels y0 + LPR n
    const int gr = tid / LPR, y0 = tid % LPR, gq = q0 + gr;
    const bool rok = gq < C;
    const unsigned woff = 4u * (unsigned)(gq * V1 + y0);                    // (past the frame: reads 0)
    const unsigned base = gq > 0 ? (unsigned)((gq - 1) % V + 1) * V : 0u;   // label y leads to state base + y
    const unsigned boff = 4u * (base + y0), boff0 = y0 == 0 ? 4u * gq : boff;
    // states in the order in which an operand of the contraction over states holds them: state r + 4 h + 8 n of the
    // accumulators' lane half h is element r + 4 (n % 2) of half h in step n / 2
    const int pos = 16 * (gr >> 4) + 8 * ((gr >> 2) & 1) + 4 * ((gr >> 3) & 1) + (gr & 3);

    struct Frame {
        float w[NS], b[NS], a;
        unsigned short f[2];                                // (bfloat16 as it came: converted when it is used)
        EmbNorm n;
    };
    auto raw_frame = [&](int i) __attribute__((always_inline)) { return a.frames[min(i, hi - 1)]; };
    auto uniform = [&](int2 v) __attribute__((always_inline)) {
        return make_int2(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y));
    };
    auto request = [&](Frame& x, int2 v) __attribute__((always_inline)) {
        const em_buf wr = em_make_buf(a.w + (size_t)v.x * fr, (unsigned)(4 * fr));
        const size_t ra = (size_t)v.x + v.y;
        const em_buf ar = em_make_buf(g.alpha + ra * C, 4u * C), br = em_make_buf(g.beta + (ra + 1) * C, 4u * C);
#pragma unroll
        for (int n = 0; n < NS; ++n) x.w[n] = em_load(wr, woff + 4u * LPR * n);
#pragma unroll
        for (int n = 0; n < NS; ++n) x.b[n] = em_load(br, (n == 0 ? boff0 : boff + 4u * LPR * n));
        x.a = em_load(ar, 4u * gq);
        x.n = g.norm[v.x];
    };
    auto request_f = [&](Frame& x, int2 v) __attribute__((always_inline)) {
        const unsigned short* f = (const unsigned short*)a.f + (size_t)v.x * H + k0;
        x.f[0] = f[0];
        x.f[1] = f[32];
    };
    // marginals of a frame -> LDS
    auto put = [&](const Frame& x, int i, int buf) __attribute__((always_inline)) {
        const bool live = i < hi && rok && x.a != LAST_NEG_INF;       // (an arc out of an unreachable state does not count, whatever its weight)
        const float al = (float)((double)x.a + x.n.k);
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            const int y = y0 + LPR * n;
            if (y <= V) {
                float v = live ? x.n.iz * em_exp(al + x.b[n] + x.w[n]) : 0.f;
                if (NUM) {
                    float* p = &s.num[buf][gr * (16 * KY + 1) + y];
                    v -= *p;
                    *p = 0.f;
                }
                if (y == 0) {
                    s.g0[buf][gr] = v;
                } else {
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const __bf16 part = (__bf16)v;
                        v -= (float)part;
                        s.g1[buf][p][gr * S1 + y - 1] = part;
                        s.g2[buf][p][(y - 1) * S2 + pos] = part;
                    }
                }
            }
        }
    };
    // cells of the intersected lattice in this tile: one a thread, in registers while the item stays the same
    int nb = -1, ncell = 0, ent = 0;
    const int* cp = nullptr;
    auto cells_of = [&](int b) __attribute__((always_inline)) {
        if (b == nb) return;
        nb = b;
        const int* st = g.starts + (size_t)b * (a.tiles + 1) + tile;
        const int c0 = __builtin_amdgcn_readfirstlane(st[0]);
        ncell = __builtin_amdgcn_readfirstlane(st[1]) - c0;
        cp = g.cells + (size_t)b * g.U1 + c0;
        ent = tid < ncell ? cp[tid] : 0;
        asm volatile("" : "+v"(ent));                      // (waited for here, not by every frame)
    };
    auto add_cell = [&](int e, float2 p, int buf) __attribute__((always_inline)) {
        float* d = &s.num[buf][((e >> 7) & 31) * (16 * KY + 1)];
        unsafeAtomicAdd(d, p.x);
        if (e & 127) unsafeAtomicAdd(d + (e & 127), p.y);
    };
    struct Num { float2 p; int ent, n; const int* cp; };
    auto request_cells = [&](Num& x, int2 v, int i) __attribute__((always_inline)) {
        cells_of(v.y);
        x.ent = ent;
        x.n = i < hi ? ncell : 0;
        x.cp = cp;
        x.p = g.pn[(size_t)v.x * g.U1 + (ent >> 12)];       // (no condition: the waits for what was requested are counted)
    };
    auto add_cells = [&](const Num& x, int2 v, int buf) __attribute__((always_inline)) {
        if (tid < x.n) add_cell(x.ent, x.p, buf);
        for (int i = tid + 64 * NW; i < x.n; i += 64 * NW) add_cell(x.cp[i], g.pn[(size_t)v.x * g.U1 + (x.cp[i] >> 12)], buf);
    };

    auto compute = [&](const float (&f)[2], int2 v, bool live, int buf) __attribute__((always_inline)) {
        float cs[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            f32x4 z[4];                                     // marginals of the empty label
#pragma unroll
            for (int n = 0; n < 4; ++n) z[n] = *(const f32x4*)&s.g0[buf][8 * n + 4 * half];
            f32x16 d;
#pragma unroll
            for (int r = 0; r < 16; ++r) d[r] = z[r >> 2][r & 3] * w0[kt];
#pragma unroll
            for (int ky = 0; ky < KY; ++ky)
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const bf16x8 gv = *(const bf16x8*)&s.g1[buf][p][(lane & 31) * S1 + 16 * ky + 8 * half];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gv, wt[kt][ky], d, 0, 0, 0);
                }
            bf16x8 g2v[2 * P];                              // (d is on the matrix cores while h is formed)
            if (KY == 2) {
#pragma unroll
                for (int k = 0; k < 2 * P; ++k) g2v[k] = *(const bf16x8*)&s.g2[buf][k % P][(lane & 31) * S2 + 16 * (k / P) + 8 * half];
            }
            u32x4 hp[2];                                    // h of the 16 states, bf16, operand order
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                float e0, e1;
                if constexpr (PAIRS) { unsigned v = ep[kt][r >> 1]; asm volatile("" : "+v"(v)); e0 = bf_lo(v); e1 = bf_hi(v); }
                else { e0 = ee[kt][r]; e1 = ee[kt][r + 1]; }
                const f32x2 p = {em_tanh(f[kt] + e0), em_tanh(f[kt] + e1)};
                hp[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2));
            }
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const bf16x8 gv = KY == 2 ? g2v[P * st + p] : *(const bf16x8*)&s.g2[buf][p][(32 * n + (lane & 31)) * S2 + 16 * st + 8 * half];
                        dw[kt][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, hp[st]), gv, dw[kt][n], 0, 0, 0);
                    }
            cs[kt] = 0.f;
            float h0 = 0.f;                                 // (a sum of its own: dw0 grows over many frames)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const unsigned pair = hp[r >> 3][(r & 7) >> 1];
                const float h = r & 1 ? bf_hi(pair) : bf_lo(pair);
                const float u = fmaf(-h, h, 1.f);
                de[kt][r] = fmaf(d[r], u, de[kt][r]);
                cs[kt] = fmaf(d[r], u, cs[kt]);
                h0 = fmaf(h, z[r >> 2][r & 3], h0);
            }
            dw0[kt] += h0;
            // (the sums are not put off to the end of the frame, where h and d of both halves would still be needed)
            asm volatile("" : "+v"(de[kt]), "+v"(dw0[kt]), "+v"(cs[kt]));
        }
        // sum over the 32 states: lanes of the other half hold the other 16; half 0 stores k0, half 1 k0 + 32
        const float send = half ? cs[0] : cs[1], keep = half ? cs[1] : cs[0];
        const float sum = keep + __shfl_xor(send, 32);
        if (live) g.pdf[((size_t)tile * a.B * a.T + v.x) * H + k0 + 32 * half] = sum;
    };

    float* pde = g.pde + ((size_t)grp * a.tiles * kEmTile + q0 + 4 * half) * H + k0;
    // dW so far, and de of a loss -> the partial sums of this workgroup
    auto flush = [&](bool first) __attribute__((always_inline)) {
        float* o = g.pdw + ((size_t)(grp * a.tiles + tile) * H + 64 * wave) * V1;
        // (no other workgroup adds to them; an addition in the L2 needs no register for the old value)
        auto add = [&](float* p, float v) __attribute__((always_inline)) {
            if (first) *p = v;
            else unsafeAtomicAdd(p, v);
        };
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int y = 32 * n + (lane & 31) + 1;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (y <= V) add(o + (size_t)(32 * kt + (r & 3) + 8 * (r >> 2) + 4 * half) * V1 + y, dw[kt][n][r]);
                dw[kt][n] = f32x16{};
            }
            const float z0 = dw0[kt] + __shfl_xor(dw0[kt], 32);
            if (half == 0) add(o + (size_t)(32 * kt + lane) * V1, z0);
            dw0[kt] = 0.f;
            if (NUM) {
#pragma unroll
                for (int r = 0; r < 16; ++r) add(pde + (size_t)((r & 3) + 8 * (r >> 2)) * H + 32 * kt, de[kt][r]);
                de[kt] = f32x16{};
            }
        }
    };

    if (lo < hi) {
        Frame x[FP];
        Num m[FP];
        int2 v0[FP], v1[FP], v2[FP], nv[FP];
        float f[FP][2];
        auto used_f = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                f[j][0] = bf_lo(x[j].f[0]);
                f[j][1] = bf_lo(x[j].f[1]);
                asm volatile("" : "+v"(f[j][0]), "+v"(f[j][1]));      // (read before the registers are requested into again)
            }
        };
#pragma unroll
        for (int j = 0; j < FP; ++j) {
            v0[j] = uniform(raw_frame(lo + j));
            v1[j] = uniform(raw_frame(lo + FP + j));
            v2[j] = uniform(raw_frame(lo + 2 * FP + j));
            nv[j] = raw_frame(lo + 3 * FP + j);
            request(x[j], v0[j]);
            request_f(x[j], v0[j]);
        }
        if (NUM) {
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                request_cells(m[j], v0[j], lo + j);
                add_cells(m[j], v0[j], j);
                request_cells(m[j], v1[j], lo + FP + j);
                add_cells(m[j], v1[j], FP + j);
                request_cells(m[j], v2[j], lo + 2 * FP + j);
            }
            em_lds_barrier();
        }
#pragma unroll
        for (int j = 0; j < FP; ++j) put(x[j], lo + j, j);
        used_f();
#pragma unroll
        for (int j = 0; j < FP; ++j) {
            request(x[j], v1[j]);
            request_f(x[j], v1[j]);
        }
        em_lds_barrier();
        // the frames from i on are used; the marginals of those after them are formed, the requests for the next ones
        // go out and their cells are added up.  dW is put away every 64 frames: a sum over a thousand frames of values
        // of which a few are near 1 and most near 1e-4 loses 2.4e-6 of it.  So is de of a loss.
        for (int i = lo; i < hi;) {
            for (const int end = min(i + 64, hi); i < end; i += FP) {
                const int cur = (i - lo) & FP ? FP : 0, nxt = FP - cur;
                int2 v3[FP];
#pragma unroll
                for (int j = 0; j < FP; ++j) {
                    v3[j] = uniform(nv[j]);                 // (requested FP frames ago)
                    nv[j] = raw_frame(i + 4 * FP + j);
                }
#pragma unroll
                for (int j = 0; j < FP; ++j) compute(f[j], v0[j], i + j < hi, cur + j);
#pragma unroll
                for (int j = 0; j < FP; ++j) put(x[j], i + FP + j, nxt + j);
                used_f();
#pragma unroll
                for (int j = 0; j < FP; ++j) {
                    request(x[j], v2[j]);
                    request_f(x[j], v2[j]);
                }
                if (NUM) {
#pragma unroll
                    for (int j = 0; j < FP; ++j) {
                        add_cells(m[j], v2[j], cur + j);
                        request_cells(m[j], v3[j], i + 3 * FP + j);
                    }
                }
#pragma unroll
                for (int j = 0; j < FP; ++j) { v0[j] = v1[j]; v1[j] = v2[j]; v2[j] = v3[j]; }
                em_lds_barrier();
            }
            flush(i <= lo + 64);
        }
    }
    if (lo >= hi) flush(true);
    if (NUM) return;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) pde[(size_t)((r & 3) + 8 * (r >> 2)) * H + 32 * kt] = de[kt][r];
}

template <int NW, int KY, bool NUM>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW > 4 ? 2 : 1, 2))) void emb_grad_kernel(EmbArgs a, EmbGradArgs g)
{
    extern __shared__ __align__(16) unsigned char em_smem[];
    typedef EmGradLds<NW, KY, NUM> S;
    S& s = *(S*)em_smem;
    for (int i = threadIdx.x; i < (int)(sizeof(S) / 4); i += 64 * NW) ((int*)em_smem)[i] = 0;
    const int tile = blockIdx.x % a.tiles, grp = blockIdx.x / a.tiles;
    const long long n = a.count[0];
    const int lo = (int)(n * grp / g.ngr), hi = (int)(n * (grp + 1) / g.ngr);
    __syncthreads();
    emb_grad_body<NW, KY, NUM>(a, g, s, tile, grp, lo, hi);
}

// the partial sums of emb_grad_kernel added up; blocks: nbf for df, nbe for de, the rest for dW (32 elements each)
__global__ __launch_bounds__(256) void emb_sum_kernel(EmbArgs a, EmbGradArgs g, int nbf, int nbe)
{
    __shared__ float red[8][32];
    const int tid = threadIdx.x, H4 = a.H / 4;
    const size_t BT = (size_t)a.B * a.T;
    struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };      // (the caller's gradients lie anywhere)
    auto write = [&](float* at, float4 v, bool add) {
        F4* p = (F4*)at;
        v = make_float4(g.scale * v.x, g.scale * v.y, g.scale * v.z, g.scale * v.w);
        if (add) {
            const F4 o = *p;
            v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
        }
        *p = F4{v.x, v.y, v.z, v.w};
    };
    auto sum4 = [&](const float4* p, size_t stride, int n) {
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
        for (int i = 0; i < n; ++i) {
            const float4 v = p[(size_t)i * stride];
            s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
        }
        return s;
    };
    const int blk = blockIdx.x;
    if (blk < nbf) {
        const size_t i = (size_t)blk * 256 + tid;
        if (i >= BT * H4) return;
        const int row = (int)(i / H4), b = row / a.T, t = row - b * a.T;
        const int L = a.len[b];
        const bool live = L <= a.T && t < L;                // (L < 0: no frame)
        if (!live && g.acc_df) return;
        write(g.df + 4 * i, live ? sum4((const float4*)g.pdf + i, BT * H4, a.tiles) : make_float4(0.f, 0.f, 0.f, 0.f), g.acc_df);
    } else if (blk < nbf + nbe) {
        const size_t i = (size_t)(blk - nbf) * 256 + tid;
        if (i >= (size_t)a.C * H4) return;
        write(g.de + 4 * i, sum4((const float4*)g.pde + i, (size_t)a.tiles * kEmTile * H4, g.ngr), g.acc_rest);
    } else {
        const int n = a.H * (a.V + 1), e = (blk - nbf - nbe) * 32 + (tid & 31), grp = tid >> 5;
        float s = 0.f;
        if (e < n) {
#pragma unroll 8
            for (int i = grp; i < a.tiles * g.ngr; i += 8) s += g.pdw[(size_t)i * n + e];
        }
        red[grp][tid & 31] = s;
        __syncthreads();
        if (tid < 32 && e < n) {
            s = red[0][tid];
            for (int k = 1; k < 8; ++k) s += red[k][tid];
            s *= g.scale;
            g.dW[e] = g.acc_rest ? g.dW[e] + s : s;
        }
    }
}

// a kernel that wants more than 64 KiB of LDS has to be told so once on every device it runs on
hipError_t em_allow_lds(const void* kernel, size_t bytes)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void*>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count({dev, kernel})) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done.insert({dev, kernel});
    return e;
}

template <typename F>
void em_label_tiles(int NT, F&& f)
{
    switch (NT) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    default: f(std::integral_constant<int, 5>()); break;
    }
}

}  // namespace

int emb_stretches(int tiles, size_t frames, int shortest, int startup)
{
    const long long most = std::max((long long)1, std::min((long long)64, (long long)(frames / (size_t)shortest)));
    long long best = 0;
    int n = 1;
    for (int ch = 1; ch <= most; ++ch) {
        const long long rounds = ((long long)tiles * ch + 255) / 256;
        const long long cost = rounds * ((long long)((frames + ch - 1) / ch) + startup);
        if (ch == 1 || cost < best) { best = cost; n = ch; }
    }
    return n;
}

EmbPlan emb_plan(int B, int T, int C, int V, int H)
{
    EmbPlan p{};
    p.tiles = (C + kEmTile - 1) / kEmTile;
    p.row = (size_t)C * (V + 1) * sizeof(float);
    p.nch = emb_stretches(p.tiles, (size_t)B * T, 8, 16);
    p.ngr = emb_stretches(p.tiles, (size_t)B * T, 16, 16);
    p.lds = (size_t)(H / 32) * (4096 + label_tiles(V) * 1024);
    p.ok = label_tiles(V) <= kEmMaxLabelTiles;
    return p;
}

hipError_t emb_launch_weights(const EmbArgs& a, const EmbPlan& p, hipStream_t st)
{
    const size_t nf = (size_t)a.B * a.T * a.H, ne = (size_t)a.C * a.H, ne_pad = (size_t)a.tiles * kEmTile * a.H;
    const int NT = label_tiles(a.V);
    hipLaunchKernelGGL(emb_prepare_kernel, dim3(kEmScan), dim3(256), 0, st, a, nf, ne, ne_pad, NT);
    hipError_t e = hipSuccess;
    em_label_tiles(NT, [&](auto N) {
        auto k = emb_weights_kernel<decltype(N)::value>;
        e = em_allow_lds((const void*)k, 159 * 1024);         // (the barrier's reduction takes a little static LDS)
        if (e == hipSuccess) hipLaunchKernelGGL(k, dim3(a.tiles * a.nch), dim3(64 * kEwWaves), p.lds, st, a);
    });
    return e != hipSuccess ? e : hipGetLastError();
}

hipError_t emb_launch_numerator(const EmbArgs& a, const EmbNumArgs& n, hipStream_t st)
{
    for (int t0 = 0; t0 < a.T; t0 += 65535)
        hipLaunchKernelGGL(emb_cell_marginals_kernel, dim3((n.U1 + 255) / 256, std::min(a.T - t0, 65535), a.B), dim3(256), 0, st, a, n, t0);
    hipLaunchKernelGGL(emb_cells_kernel, dim3(a.B), dim3(256), (size_t)(a.tiles + 1) * sizeof(int), st, a, n);
    return hipGetLastError();
}

hipError_t emb_launch_gradient(const EmbArgs& a, const EmbGradArgs& g, hipStream_t st)
{
    const size_t rows = (size_t)a.B * a.T;
    hipLaunchKernelGGL(emb_norm_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, a, g);
    hipError_t e = hipSuccess;
    auto launch = [&](auto NW, auto KY, auto NUM) {
        constexpr int nw = decltype(NW)::value, ky = decltype(KY)::value;
        constexpr bool num = decltype(NUM)::value;
        constexpr size_t lds = sizeof(EmGradLds<nw, ky, num>);
        static_assert(2 * lds <= 160 * 1024, "two workgroups of few waves a compute unit");
        auto k = emb_grad_kernel<nw, ky, num>;
        e = em_allow_lds((const void*)k, lds);
        if (e == hipSuccess) hipLaunchKernelGGL(k, dim3(a.tiles * g.ngr), dim3(64 * nw), lds, st, a, g);
    };
    auto go = [&](auto NW, auto KY) {
        if (g.pn) launch(NW, KY, std::true_type());
        else launch(NW, KY, std::false_type());
    };
    auto steps = [&](auto NW) {
        if (grad_steps(a.V) == 2) go(NW, std::integral_constant<int, 2>());
        else go(NW, std::integral_constant<int, 4>());
    };
    switch (a.H / 64) {
    case 2: steps(std::integral_constant<int, 2>()); break;
    case 4: steps(std::integral_constant<int, 4>()); break;
    case 6: steps(std::integral_constant<int, 6>()); break;
    default: steps(std::integral_constant<int, 8>()); break;
    }
    if (e != hipSuccess) return e;
    const unsigned nbf = (unsigned)((rows * (a.H / 4) + 255) / 256), nbe = (unsigned)(((size_t)a.C * (a.H / 4) + 255) / 256);
    const unsigned nbw = (unsigned)((a.H * (a.V + 1) + 31) / 32);
    hipLaunchKernelGGL(emb_sum_kernel, dim3(nbf + nbe + nbw), dim3(256), 0, st, a, g, (int)nbf, (int)nbe);
    return hipGetLastError();
}

}  // namespace last
