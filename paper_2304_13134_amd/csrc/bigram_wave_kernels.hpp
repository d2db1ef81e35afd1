// Full 1-gram contexts of up to 64 labels with dense weights: the recursions of Eq. 2 (arXiv 2304.13134)
// in both directions and the tropical one (Section 4.2.3), one workgroup per item and direction, the whole
// chain of frames in the registers of ONE wavefront.
//
// What bounds these shapes is the chain of a frame, not its 4 to 17 KB.  With the rows dealt out to several waves
// that chain was readlanes, partial sums through LDS, a barrier and a normalisation: 0.72 us a frame at 32 labels, 0.54 us
// tropical.  Here
//  - a frame is one matrix-vector product of V x V label states (the start state, which nothing leads back to, goes apart)
//    in fused multiply-adds whose state operand is broadcast by the instruction itself (DPP row_newbcast: lane k of
//    each row of sixteen to the whole row).  Each row of sixteen lanes keeps a share of the states, so that a column's sum is
//    spread over the four rows and two lane swaps bring it back to the lanes that hold the states: 16
//    multiply-adds a frame up to 32 labels (BwNarrow), 48 or 64 beyond (BwWide), no LDS and no barrier on the chain;
//  - the scale of a frame's vector is chosen a frame ahead from the largest state before and the largest shift of the frame,
//    an upper bound, so that the maximum over the lanes is off the chain.  A frame whose vector comes out too small
//    under that bound (2^12 of room for differences between the rows' largest weights) is scaled exactly;
//  - eight waves ("producers") fetch the weights of a group of frames with 16-byte loads two groups ahead and turn them into
//    E = 2^(w log2 e - s_q) <= 1, s_q >= max_y w[q][y] log2 e an integer per row, in LDS (backward: transposed), while the chain
//    works on the group before; a ninth takes the start state's rows of all frames of the group.  One barrier a group.
//    Every lane of a row instruction has a piece (LPR lanes a row, RPI rows an instruction).
// Tropical: the weights as they are, sums and maxima in the same places; the chain keeps no backpointers but stores the vector
// of every frame, and bigram_bp_kernel finds the sources of all frames at once: the same float32 sums, compared exactly.
//
// Arithmetic is scaled linear float32: x_q = 2^(s_q - S) state_q with the largest of them in [2^100, 2^120), S adds up
// in a float64 offset per frame.  What is lost is what lies 2^126 below the largest weight of its row or 2^226
// below the largest state of its frame: nothing to a sum, unless paths make up for it elsewhere.  With marginals an item
// that may have lost a part is flagged (marginals_kernels.hpp); for a distance alone the chain takes notes and
// bigram_join_kernel computes such items again (see bigram_kernels.hpp; the thresholds here are relative to the
// largest state).
#pragma once
#include "bigram_kernels.hpp"

namespace last {

constexpr int kBwProducers = 8;
constexpr int kBwThreads = (kBwProducers + 2) * kWave;
constexpr int kBwMaxV = 64;
constexpr int kBwRoom = 112;             // S = exponent of the largest state + largest shift - kBwRoom: sums of 66 stay below 2^127
constexpr float kBwLow = 1.2676506e30f;  // 2^100
constexpr int kBwNone = -0x10000000;     // shift of a place without a state

// Places of the label states: the last 16-byte piece of a row ends with the row, so where V is no multiple of four
// the last four labels are at the last four places and some places before them are copies without a state.
__device__ __forceinline__ int bw_label(int place, int V)           // label - 1
{
    const int P = (V + 3) & ~3;
    return max(0, min(place < P - 4 || V < 4 ? place : place - (P - V), V - 1));
}
__device__ __forceinline__ bool bw_valid(int place, int V)
{
    const int P = (V + 3) & ~3;
    return V < 4 ? place < V : place < P - 4 || (place < P && place - (P - V) >= P - 4);
}

// Up to 32 labels.  Lane (j, i) of the wave (row j of sixteen) sums columns 2i, 2i+1 over the states 2(k + 8(j/2)) + j%2, k < 8.
template <int U_>
struct BwNarrow {
    static constexpr int U = U_;         // row instructions of a producer and frame: 8 U >= V rows
    static constexpr int CPL = 2, KB = 8, N = 32, LPR = 8, RPI = 8, G = 8, WPF = 1;
    static constexpr int Pitch = 36, PitchB = 34;
    static constexpr bool All = U == 4;  // the producers write every place
    static __device__ __forceinline__ int place(int lane) { return 2 * (((lane & 15) + ((lane >> 5) << 3)) & 15) + ((lane >> 4) & 1); }
    static __device__ __forceinline__ int first_row(int lane) { return 16 * (lane >> 5) + ((lane >> 4) & 1); }
    static constexpr int RowStep = 2;
};
// 33 to 4 KB labels.  Lane (j, i) sums columns 4i .. 4i+3 over the states 4k + j.
template <int KB_>
struct BwWide {
    static constexpr int KB = KB_, U = KB_ / 2;
    static constexpr int CPL = 4, N = 4 * KB_, LPR = 16, RPI = 4, G = 4, WPF = 2;
    static constexpr int Pitch = 68, PitchB = 68;
    static constexpr bool All = KB == 16;
    static __device__ __forceinline__ int place(int lane) { return 4 * (lane & 15) + (lane >> 4); }
    static __device__ __forceinline__ int first_row(int lane) { return lane >> 4; }
    static constexpr int RowStep = 4;
};
// a frame in LDS
template <typename D>
struct BwFrame {
    float E[D::N * D::Pitch];
    struct { float est, unused, e0; int sh; } st[64];     // by place: start state's row, empty label, row shift
    int hdr[4];                          // largest shift of each producer's rows; start state: shift, E of its empty label
};

// acc[c] += sum_k x[lane k of the row] E[k][c].  In one piece, because an instruction that reads a lane of a register must
// not follow within two others that one which wrote it, and neither may a lane swap: the compiler does not look inside.
template <int KB>
__device__ __forceinline__ void bw_sum(float x, const float (&E)[KB][2], float (&acc)[2])
{
    static_assert(KB == 8, "one block");
    float a0, a1, b0, b1;
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %4, %5 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %1, %4, %6 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %2, %4, %7 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %3, %4, %8 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %9 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %10 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %4, %11 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %4, %12 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %13 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %14 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %4, %15 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %4, %16 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %17 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %18 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %4, %19 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %4, %20 row_newbcast:7 row_mask:0xf bank_mask:0xf"
        : "=&v"(a0), "=&v"(a1), "=&v"(b0), "=&v"(b1)
        : "v"(x), "v"(E[0][0]), "v"(E[0][1]), "v"(E[1][0]), "v"(E[1][1]), "v"(E[2][0]), "v"(E[2][1]), "v"(E[3][0]), "v"(E[3][1]),
          "v"(E[4][0]), "v"(E[4][1]), "v"(E[5][0]), "v"(E[5][1]), "v"(E[6][0]), "v"(E[6][1]), "v"(E[7][0]), "v"(E[7][1]));
    acc[0] = a0 + b0;
    acc[1] = a1 + b1;
}
// Four columns a lane: the broadcast as a move of its own (in every addition of the tropical recursion 0.36 us a frame
// of 47 labels instead of 0.33; with two columns a lane it is the other way round, 0.206 against 0.219 at 32).
template <int K>
__device__ __forceinline__ float bw_bcast(float x)      // lane K of the lane's row of sixteen
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + K, 0xf, 0xf, true));
}
template <int KB, int K = 0>
__device__ __forceinline__ void bw_sum(float x, const float (&E)[KB][4], float (&acc)[4])
{
    const float q = bw_bcast<K>(x);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = K == 0 ? q * E[K][c] : fmaf(q, E[K][c], acc[c]);
    if constexpr (K + 1 < KB) bw_sum<KB, K + 1>(x, E, acc);
}
// acc[c] = max over k of x[lane k of the row] + E[k][c]
template <int KB, int CPL, int K = 0>
__device__ __forceinline__ void bw_max(float x, const float (&E)[KB][CPL], float (&acc)[CPL])
{
    const float q0 = bw_bcast<K>(x), q1 = bw_bcast<K + 1>(x);
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        acc[c] = c3_max3(K == 0 ? LAST_NEG_INF : acc[c], __fadd_rn(q0, E[K][c]), __fadd_rn(q1, E[K + 1][c]));
    if constexpr (K + 2 < KB) bw_max<KB, CPL, K + 2>(x, E, acc);
}
template <bool MAX>
__device__ __forceinline__ float bw_op(float x, float y) { return MAX ? v3_fmax(x, y) : x + y; }
template <bool MAX>
__device__ __forceinline__ float bw_merge16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return bw_op<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <bool MAX>
__device__ __forceinline__ float bw_merge32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return bw_op<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// column sums (maxima), spread over the four rows of lanes -> the lanes that hold the states
template <bool MAX>
__device__ __forceinline__ float bw_home(const float (&a)[2])
{
    const float u = bw_merge16<MAX>(a[0], a[1]);             // rows of lanes: columns 2i, 2i + 1, 2i, 2i + 1
    const float v = bw_merge32<MAX>(u, u);
    return dpp_f<0x128, 0xc>(v, v);                          // the upper half keeps the upper half of the states in lanes 0 .. 7
}
template <bool MAX>
__device__ __forceinline__ float bw_home(const float (&a)[4])
{
    return bw_merge16<MAX>(bw_merge32<MAX>(a[0], a[2]), bw_merge32<MAX>(a[1], a[3]));
}
// v[lane] = x for a lane that is a constant once the group is unrolled
__device__ __forceinline__ void bw_writelane(int& v, int x, int lane)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "i"(lane));
}
template <int N>
__device__ __forceinline__ int bw_ror(int x) { return __builtin_amdgcn_mov_dpp(x, 0x120 + N, 0xf, 0xf, true); }
template <int N>
__device__ __forceinline__ float bw_ror(float x) { return __int_as_float(bw_ror<N>(__float_as_int(x))); }
// largest of the lanes' non-negative floats, as bits
template <bool WIDE>
__device__ __forceinline__ unsigned bw_top_bits(int m)
{
    m = max(m, bw_ror<8>(m));
    m = max(m, bw_ror<4>(m));
    m = max(m, bw_ror<2>(m));
    m = max(m, bw_ror<1>(m));
    int r = max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16));
    if (WIDE) r = max(r, max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
    return (unsigned)r;
}

// largest of each aligned group of 8 (sixteen: 16) lanes, in all of them, for a few rows at a time: two instructions
// between the write of a register and the read of its lanes
__device__ __forceinline__ void bw_row_max(float (&m)[1], bool sixteen)
{
    if (sixteen)
        asm("s_nop 1\n\t"
            "v_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "" : "+v"(m[0]));
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "" : "+v"(m[0]));
}
__device__ __forceinline__ void bw_row_max(float (&m)[2], bool sixteen)
{
    if (sixteen)
        asm("s_nop 1\n\t"
            "v_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_max_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "" : "+v"(m[0]), "+v"(m[1]));
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "" : "+v"(m[0]), "+v"(m[1]));
}
__device__ __forceinline__ void bw_row_max(float (&m)[4], bool sixteen)
{
    if (sixteen)
        asm("s_nop 1\n\t"
            "v_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_max_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_max_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_max_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
            "" : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]));
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %3, %3, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_max_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "" : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]));
}
template <int N>
__device__ __forceinline__ void bw_row_max(float (&m)[N], bool sixteen)
{
    static_assert(N == 6 || N == 8, "");
    float a[4] = {m[0], m[1], m[2], m[3]}, b[N - 4];
#pragma unroll
    for (int i = 4; i < N; ++i) b[i - 4] = m[i];
    bw_row_max(a, sixteen);
    bw_row_max(b, sixteen);
#pragma unroll
    for (int i = 0; i < N; ++i) m[i] = i < 4 ? a[i] : b[i - 4];
}

// grid (B, roles): blockIdx.y = 0 forward, 1 backward.  Dynamic LDS: two groups of G frames.
// KEEP: every row at [b][T+1][C], distance written; else the meeting row at [b][C].
// Tropical: bp (may be null) receives the bits of the vector before frame t in row t (see bigram_bp_kernel).
template <typename D, bool TROP, bool KEEP>
__global__ __launch_bounds__(kBwThreads) void bigram_wave_kernel(BiArgs a)
{
    constexpr int CPL = D::CPL, KB = D::KB, U = D::U, G = D::G, LPR = D::LPR, RPI = D::RPI;
    constexpr bool WIDE = CPL == 4;
    typedef BwFrame<D> F;
    extern __shared__ __align__(16) unsigned char bw_s[];
    F* const ring = (F*)bw_s;                                  // [2][G]
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool back = !TROP && blockIdx.y == 1;
    const int C = a.C, V = C - 1, L = a.len[b];
    if (L < 0 || L > a.T) {
        if ((TROP || KEEP) && !back && tid == 0) {
            a.dist[b] = __builtin_nanf("");
            if (!TROP) a.D2[b] = __builtin_nan("");
            if (TROP && a.final_state) a.final_state[b] = -1;
            if (a.item_status) a.item_status[b] = kItemBadLength;
        }
        return;
    }
    const int low = KEEP ? 1 : L / 2;
    const int steps = TROP ? L : back ? max(L - low, 0) : KEEP ? L : L / 2;
    const int groups = ((steps + G - 1) / G + 1) & ~1;       // (pairs: what the last of them has too many is not used)
    if (!D::All) {
        // places that no producer writes: zero weights of no state
        for (int i = tid; i < (int)(2 * G * sizeof(F) / 16); i += kBwThreads) ((float4*)bw_s)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        __syncthreads();
        for (int i = tid; i < 2 * G * 64; i += kBwThreads) ring[i >> 6].st[i & 63].sh = kBwNone;
    }
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;

    auto produce = [&](auto BK) __attribute__((always_inline)) {
        // ------------------------------------------------------------ producers
        constexpr bool BACK = decltype(BK)::value;
        // (waves go to the SIMDs in turn: the chain's has the light ninth producer, wave 4, and one other)
        const bool first_row = wave == 4;
        const int p = wave < 4 ? wave - 1 : wave - 2;           // 0 .. 7
        const int lq = lane / LPR, lc = lane - lq * LPR;
        const int fi = p / D::WPF, half = first_row ? 0 : p % D::WPF;      // (uniform: descriptors are made of them)
        const int c0 = V < 4 ? 0 : min(4 * lc, V - 4);
        const size_t fr = (size_t)C * C;
        const float* wi = a.w + (size_t)b * a.T * fr;
        const unsigned frb = 4u * (unsigned)fr;
        auto place_of = [&](int u) __attribute__((always_inline)) { return RPI * (half * U + u) + lq; };
        unsigned voff[U], boff;
#pragma unroll
        for (int u = 0; u < U; ++u) voff[u] = 4u * (unsigned)((1 + bw_label(place_of(u), V)) * C + 1 + c0);
        // the empty label of row u comes with lane u of the row
        boff = lc < U ? 4u * (unsigned)((1 + bw_label(place_of(min(lc, U - 1)), V)) * C) : 0xfffffff0u;
        if (first_row) {
            voff[0] = 4u * (unsigned)(1 + c0);
            boff = lc == 0 ? 0u : 0xfffffff0u;
        }
        auto frame_ptr = [&](int n) __attribute__((always_inline)) {
            const int t = BACK ? max(L - 1 - n, 0) : min(n, L - 1);
            return wi + (size_t)t * fr;
        };
        // fewer than four labels (tropical only): what a piece holds past the row is no arc
        auto few = [&](float4& w) __attribute__((always_inline)) {
            w.y = V < 2 ? LAST_NEG_INF : w.y;
            w.z = V < 3 ? LAST_NEG_INF : w.z;
            w.w = V < 4 ? LAST_NEG_INF : w.w;
        };
        float4 raw[2][U];
        float bl[2];
        if (first_row) {
            // one frame a group of LPR lanes: addresses differ within the wave
            auto issue = [&](auto S, int g) __attribute__((always_inline)) {
                const float* f = frame_ptr(g * G + lq);
                struct __attribute__((packed, aligned(4))) f4 { float v[4]; };
                // (fewer than four labels: the whole frame is 16 floats at most and the piece may reach past it)
                f4 v;
                if (V >= 4) v = *(const f4*)(f + 1 + c0);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v.v[e] = f[1 + min(e, V - 1)];
                }
                raw[decltype(S)::value][0] = make_float4(v.v[0], v.v[1], v.v[2], v.v[3]);
                bl[decltype(S)::value] = f[0];
            };
            auto prep = [&](auto S, int g) __attribute__((always_inline)) {
                constexpr int Z = decltype(S)::value;
                F* o = ring + (g & 1) * G + lq;
                float4 w = raw[Z][0];
                float w0 = bl[Z];
                if (TROP) few(w);
                int sh = 0;
                if (!TROP) {
                    float m[1] = {v3_fmax(c3_max3(w.x, w.y, w.z), v3_fmax(w.w, w0))};
                    bw_row_max(m, LPR == 16);
                    sh = shift_for(m[0]);
                    const float ns = -(float)sh;
                    w.x = fast_exp2(fmaf(w.x, kLog2e, ns));
                    w.y = fast_exp2(fmaf(w.y, kLog2e, ns));
                    w.z = fast_exp2(fmaf(w.z, kLog2e, ns));
                    w.w = fast_exp2(fmaf(w.w, kLog2e, ns));
                    w0 = fast_exp2(fmaf(w0, kLog2e, ns));
                }
                o->st[4 * lc].est = w.x;
                o->st[4 * lc + 1].est = w.y;
                o->st[4 * lc + 2].est = w.z;
                o->st[4 * lc + 3].est = w.w;
                if (lc == 0) {
                    o->hdr[2] = sh;
                    o->hdr[3] = __float_as_int(w0);
                    if (D::WPF == 1) o->hdr[1] = kBwNone;
                }
                issue(S, g + 2);
            };
            if (groups > 0) { issue(I0(), 0); issue(I1(), 1); }
            __syncthreads();
            for (int g = 0; g < groups; g += 2) {
                prep(I0(), g);
                lds_only_barrier();
                prep(I1(), g + 1);
                lds_only_barrier();
            }
            return;
        }
        auto issue = [&](auto S, int g) __attribute__((always_inline)) {
            const buf_t rs = make_buf(frame_ptr(g * G + fi), frb);
#pragma unroll
            for (int u = 0; u < U; ++u) raw[decltype(S)::value][u] = tri_load4(rs, voff[u], 0);
            bl[decltype(S)::value] = buf_load(rs, boff, 0);
        };
        auto prep = [&](auto S, int g) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            F* o = ring + (g & 1) * G + fi;
            const float w0 = bl[Z];
            int own = kBwNone;
            float m[U];
            if (!TROP) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float4 w = raw[Z][u];
                    m[u] = v3_fmax(c3_max3(w.x, w.y, w.z), v3_fmax(w.w, lc == u ? w0 : LAST_NEG_INF));
                }
                bw_row_max(m, LPR == 16);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float4 w = raw[Z][u];
                if (TROP) few(w);
                if (!TROP) {
                    const int sh = shift_for(m[u]);
                    own = lc == u ? sh : own;
                    const float ns = -(float)sh;
                    w.x = fast_exp2(fmaf(w.x, kLog2e, ns));
                    w.y = fast_exp2(fmaf(w.y, kLog2e, ns));
                    w.z = fast_exp2(fmaf(w.z, kLog2e, ns));
                    w.w = fast_exp2(fmaf(w.w, kLog2e, ns));
                }
                const int r = place_of(u);
                if (!BACK) {
                    *(float4*)(o->E + r * D::Pitch + 4 * lc) = w;
                } else if (4 * lc < D::N) {
                    // transposed; BwWide: sixteen rows further on the places move by four, so that the lanes of
                    // a store fall on all banks
                    const int at = 4 * lc * D::PitchB + (WIDE ? r ^ (4 * (lc >> 2)) : r);
                    o->E[at] = w.x;
                    o->E[at + D::PitchB] = w.y;
                    o->E[at + 2 * D::PitchB] = w.z;
                    o->E[at + 3 * D::PitchB] = w.w;
                }
            }
            if (lc < U) {
                const int r = place_of(lc);
                const float e0 = TROP ? w0 : fast_exp2(fmaf(w0, kLog2e, -(float)own));
                *(float2*)&o->st[r].e0 = make_float2(e0, __int_as_float(bw_valid(r, V) ? own : kBwNone));
            }
            if (!TROP) {
                const int top = wave_max_dpp(own);
                if (lane == 0) o->hdr[half] = top;
            }
            issue(S, g + 2);             // (not before: the requests would go to other registers and be waited for where they are moved)
        };
        if (groups > 0) { issue(I0(), 0); issue(I1(), 1); }
        __syncthreads();
        for (int g = 0; g < groups; g += 2) {
            prep(I0(), g);
            lds_only_barrier();
            prep(I1(), g + 1);
            lds_only_barrier();
        }
    };
    if (wave != 0) {
        if constexpr (TROP) produce(std::false_type());
        else if (back) produce(std::true_type());
        else produce(std::false_type());
        return;
    }

    // ---------------------------------------------------------------- the chain
    __builtin_amdgcn_s_setprio(3);
    __syncthreads();
    const int place = D::place(lane);
    const bool mine = bw_valid(place, V);                       // (BwNarrow: the upper half of the wave has copies)
    const bool single = mine && (WIDE || lane < 32);
    const int state = 1 + bw_label(place, V);
    const unsigned soff = single ? 4u * (unsigned)state : 0xfffffff0u;     // dropped by the range check
    const unsigned rowb = 4u * (unsigned)C;
    // the start state goes with lane 32 of the same store (BwNarrow) or lane 0 of another
    const unsigned soff0 = WIDE ? (lane == 0 ? 0u : 0xfffffff0u) : lane == 32 ? 0u : soff;

    struct Regs {
        float E[KB][CPL];
        float est, e0;
        int sh;
    };
    // A group is unrolled, and what is the same for all lanes is fetched once a group, frame f's in lane f: the wave issues an
    // instruction every five clocks or so whatever its kind, and address arithmetic was a third of a frame.
    auto run = [&](auto BK) __attribute__((always_inline)) {
        constexpr bool BACK = decltype(BK)::value;
        constexpr int Pitch = BACK ? D::PitchB : D::Pitch;
        const int i4 = lane & 15;
        const int rbase = D::first_row(lane) * Pitch;
        auto fetch = [&](Regs& x, const F* f) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                if constexpr (CPL == 2) {
                    const float2 v = *(const float2*)(f->E + rbase + 2 * i4 + k * D::RowStep * Pitch);
                    x.E[k][0] = v.x; x.E[k][1] = v.y;
                } else {
                    const int at = BACK ? rbase + 4 * (i4 ^ (k >> 2)) : rbase + 4 * i4;
                    const float4 v = *(const float4*)(f->E + at + k * D::RowStep * Pitch);
                    x.E[k][0] = v.x; x.E[k][1] = v.y; x.E[k][2] = v.z; x.E[k][3] = v.w;
                }
            }
            const float4 c = *(const float4*)&f->st[place];
            x.est = c.x;
            x.e0 = c.z;
            x.sh = __float_as_int(c.w);
        };
        int smaxv = 0, s0v = 0, e00v = 0;
        // frame(registers, number of the frame in its group): the group from frame n0 on begins with begin(n0)
        auto chain = [&](auto&& begin, auto&& frame, auto&& end) __attribute__((always_inline)) {
            Regs R[2];
            for (int g = 0; g < groups; ++g) {
                lds_only_barrier();
                const F* const f0 = ring + (g & 1) * G;
                const int nf = min(G, steps - g * G);
                if (nf <= 0) break;                                  // (the last barrier is this one)
                fetch(R[0], f0);
                const int4 h = *(const int4*)f0[lane & (G - 1)].hdr;
                smaxv = max(max(h.x, h.y), h.z);
                s0v = h.z;
                e00v = h.w;
                begin(g * G, nf);
#pragma unroll
                for (int f = 0; f < G; ++f) {
                    if (f >= nf) break;
                    if (f + 1 < G) fetch(R[(f + 1) & 1], f0 + f + 1);
                    frame(R[f & 1], f);
                }
                end(g * G, nf);
            }
        };
        auto put = [&](float x, float x0, buf_t o, unsigned so) __attribute__((always_inline)) {
            if (!WIDE) {
                buf_store(lane == 32 ? x0 : x, o, soff0, so);
            } else {
                buf_store(x, o, soff, so);
                buf_store(x0, o, soff0, so);
            }
        };
        if constexpr (TROP) {
            float v = LAST_NEG_INF, v0 = 0.f;
            const float lim = mine ? __builtin_huge_valf() : LAST_NEG_INF;
            buf_t o;
            chain([&](int t0, int nf) __attribute__((always_inline)) {
                o = make_buf(a.bp + ((size_t)b * a.T + t0) * C, a.bp ? rowb * (unsigned)nf : 0u);
            }, [&](const Regs& x, int f) __attribute__((always_inline)) {
                put(v, v0, o, rowb * (unsigned)f);
                float acc[CPL];
                bw_max<KB, CPL>(v, x.E, acc);
                const float s = c3_max3(__fadd_rn(v, x.e0), __fadd_rn(v0, x.est), LAST_NEG_INF);
                const float n = v3_fmax(bw_home<true>(acc), s);
                v = n < lim ? n : lim;
                v0 = __fadd_rn(v0, __int_as_float(__builtin_amdgcn_readlane(e00v, f)));
            }, [](int, int) {});
            // best final state, lowest index among equals
            float best = single ? v : LAST_NEG_INF;
            int idx = single ? state : 0x7fffffff;
            if (v0 >= best) { best = v0; idx = 0; }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float ov = __shfl_xor(best, o, kWave);
                const int oi = __shfl_xor(idx, o, kWave);
                if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
            }
            if (lane == 0) {
                a.dist[b] = best;
                if (a.final_state) a.final_state[b] = idx;
                if (a.item_status) a.item_status[b] = kItemOk;
            }
        } else {
            float* const base = BACK ? a.beta : a.alpha;
            double* const off = BACK ? a.offb : a.offa;
            double A = 0.0;                      // offset of the group's first frame; rel: of the frame at hand to that
            int rel = 0, relv = 0;
            unsigned back0 = 0;
            buf_t rows;
            // one row and its offset
            auto put_row = [&](float x, float x0, int t, double at) __attribute__((always_inline)) {
                const size_t row = KEEP ? (size_t)b * (a.T + 1) + t : (size_t)b;
                put(x, x0, make_buf(base + row * C, rowb), 0);
                nw_store64(at, make_buf(off + row, 8u), lane == 0 ? 0u : 0xfffffff0u, 0);
            };
            auto ended = [&](size_t first, int nf, bool down) __attribute__((always_inline)) {      // offsets of a group's rows, lane f <-> frame f
                if (KEEP && lane < nf) off[down ? first - lane : first + lane] = A + (double)relv;
                A += (double)rel;
            };
            // what a distance alone notes (see bigram_kernels.hpp)
            bool was_thin = false, unburied = false, unburied_small = false, none = false;      // none: a score is no number, nor is the sum then
            const float not_thin = mine ? 0.f : __builtin_inff();
            const unsigned not_small = mine ? 0u : ~0u;
            unsigned small = ~0u, small0 = ~0u;
            auto look = [&](float v, float v0, int M) __attribute__((always_inline)) {      // at the new states; M: of those they came from
                float least = v + not_thin;
                if (BACK) least = fminf(least, v0);
                if (!__any(least < __builtin_ldexpf(1.f, M - 40))) {
                    was_thin = false;
                    return;
                }
                unsigned s0 = small;
                if (BACK) s0 = min(s0, small0);
                unburied = unburied || was_thin;
                unburied_small = unburied_small || __any(s0 < kBiSmall);
                was_thin = __any(least < __builtin_ldexpf(1.f, M - 90));
            };
            // x = 2^(sh - S) v; S is exact where the bound was too high
            auto scale = [&](float v, float v0, int sh, int s0, int& S, float& x, float& x0) __attribute__((always_inline)) {
                x = __builtin_ldexpf(v, sh - S);
                x0 = __builtin_ldexpf(v0, s0 - S);
                if (__builtin_expect(!__any(max(__float_as_int(x), __float_as_int(x0)) >= __float_as_int(kBwLow)), 0)) {
                    int top = mine && v > 0.f ? float_exponent(v) + sh : -0x40000000;
                    if (v0 > 0.f) top = max(top, float_exponent(v0) + s0);
                    top = wave_max_dpp(top);
                    if (top == -0x40000000) top = 0;             // no state reachable
                    S = top - kBiCentre;
                    x = __builtin_ldexpf(v, sh - S);
                    x0 = __builtin_ldexpf(v0, s0 - S);
                }
            };
            auto note_small = [&](float v, float v0, int sh, int s0, int S, int M, int Mbefore, int smax) __attribute__((always_inline)) {
                if (KEEP) return;
                const int top = S + M;
                const int ex = v > 0.f ? float_exponent(v) + sh : -0x40000000;
                const int ex0 = v0 > 0.f ? float_exponent(v0) + s0 : -0x40000000;
                small = (unsigned)(ex - (top - (int)kBiAbsent)) | not_small;
                small0 = (unsigned)(ex0 - (top - (int)kBiAbsent));
                unburied = unburied || (was_thin && smax - top + Mbefore > kBiOver);
            };
            // Exponent of the largest state of the vector at hand, or more: it is looked at in every second frame (without
            // marginals in all) and stays below 120 by the choice of S.
            int M = BACK ? kBiCentre : 0;
            auto top_of = [&](float x, float x0, int f) __attribute__((always_inline)) {
                return KEEP && (f & 1) ? 119 : float_exponent(__uint_as_float(bw_top_bits<WIDE>(max(__float_as_int(x), __float_as_int(x0)))));
            };
            if constexpr (!BACK) {
                float v = 0.f, v0 = 1.f;
                chain([&](int t0, int nf) __attribute__((always_inline)) {
                    rows = make_buf(base + ((size_t)b * (a.T + 1) + t0) * C, KEEP ? rowb * (unsigned)nf : 0u);
                    rel = relv = 0;
                }, [&](const Regs& r, int f) __attribute__((always_inline)) {
                    const int smax = __builtin_amdgcn_readlane(smaxv, f), s0 = __builtin_amdgcn_readlane(s0v, f);
                    int S = M + smax - kBwRoom;
                    float x, x0;
                    scale(v, v0, r.sh, s0, S, x, x0);
                    if (KEEP) {
                        put(v, v0, rows, rowb * (unsigned)f);
                        bw_writelane(relv, rel, f);
                    }
                    rel += S;
                    float acc[CPL];
                    bw_sum<KB>(x, r.E, acc);
                    const int Mb = M;
                    M = top_of(x, x0, f);
                    note_small(v, v0, r.sh, s0, S, M, Mb, smax);
                    v = fmaf(x0, r.est, fmaf(x, r.e0, bw_home<false>(acc)));
                    v0 = x0 * __int_as_float(__builtin_amdgcn_readlane(e00v, f));
                    if (!KEEP) look(v, v0, M);
                }, [&](int t0, int nf) __attribute__((always_inline)) { ended((size_t)b * (a.T + 1) + t0, nf, false); });
                put_row(v, v0, steps, A);
                none = __any(v != v) || v0 != v0;
                if (KEEP) {
                    // all states of the last frame are final with weight 0
                    double z = single ? (double)v : 0.0;
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
                    if (lane == 0) {
                        const double d2 = A + log2(z + (double)v0);
                        a.D2[b] = d2;
                        a.dist[b] = (float)(d2 * 0.6931471805599453);
                        if (a.item_status) a.item_status[b] = kItemOk;
                    }
                }
            } else {
                float x = mine ? __builtin_ldexpf(1.f, kBiCentre) : 0.f, x0 = __builtin_ldexpf(1.f, kBiCentre);
                A = -(double)kBiCentre;
                if (KEEP || steps == 0) put_row(x, x0, L, A);
                chain([&](int n0, int nf) __attribute__((always_inline)) {
                    // rows L - 1 - n0 downwards
                    rows = make_buf(base + ((size_t)b * (a.T + 1) + (L - n0 - nf)) * C, KEEP ? rowb * (unsigned)nf : 0u);
                    back0 = rowb * (unsigned)(nf - 1);
                    rel = relv = 0;
                }, [&](const Regs& r, int f) __attribute__((always_inline)) {
                    const int smax = __builtin_amdgcn_readlane(smaxv, f), s0 = __builtin_amdgcn_readlane(s0v, f);
                    int S = M + smax - kBwRoom;
                    float acc[CPL];
                    bw_sum<KB>(x, r.E, acc);
                    // the start state: a sum over all lanes that hold a state (off the chain)
                    float z = x * r.est;
                    z += bw_ror<8>(z);
                    z += bw_ror<4>(z);
                    z += bw_ror<2>(z);
                    z += bw_ror<1>(z);
                    z = bw_merge16<false>(z, z);
                    if (WIDE) z = bw_merge32<false>(z, z);
                    const float v = fmaf(x, r.e0, bw_home<false>(acc));
                    const float v0 = fmaf(x0, __int_as_float(__builtin_amdgcn_readlane(e00v, f)), z);
                    if (!KEEP) look(v, v0, M);
                    scale(v, v0, r.sh, s0, S, x, x0);
                    rel += S;
                    const int Mb = M;
                    M = top_of(x, x0, f);
                    note_small(v, v0, r.sh, s0, S, M, Mb, smax);
                    if (KEEP) {
                        put(x, x0, rows, back0 - rowb * (unsigned)f);
                        bw_writelane(relv, rel, f);
                    }
                }, [&](int n0, int nf) __attribute__((always_inline)) { ended((size_t)b * (a.T + 1) + (L - 1 - n0), nf, true); });
                if (!KEEP && steps > 0) put_row(x, x0, L - steps, A);
                none = __any(x != x) || x0 != x0;
            }
            if (!KEEP) {
                const int f = none ? 0 : (unburied ? 1 : 0) | (unburied_small ? 2 : 0);
                if (lane == 0) a.wide[(size_t)b * 2 + (BACK ? 1 : 0)] = f;
            }
        }
    };
    if constexpr (TROP) run(std::false_type());
    else {
        if (back) run(std::true_type());
        else run(std::false_type());
    }
}

// Backpointers of a segment of S frames from the vectors that the tropical chain stored in their place (row t: bits of the
// scores before frame t), and the map of the segment for the backtrace: state at its upper end -> state at its lower
// end.  Candidates are the chain's own float32 sums, so the best of them is the state's score exactly; among
// equals the lowest flat arc index wins.  One wave a frame, a lane a state; kBpRows frames between barriers.
constexpr int kBpWaves = 16, kBpRows = 32;
__global__ __launch_bounds__(kBpWaves * kWave) void bigram_bp_kernel(const float* __restrict__ w, const int* __restrict__ len, int C, int T,
                                                                    int S, int nseg, int* __restrict__ bp, int* __restrict__ map)
{
    __shared__ unsigned char prev[kBpRows][kBwMaxV + 1];
    const int seg = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = len[b];
    if (L < 0 || L > T) return;
    const int t0 = seg * S, t1 = min(t0 + S, L);
    if (t0 >= t1) return;
    int q = min(tid, C - 1);                                    // threads < C: the state that theirs goes back to
    for (int hi = t1; hi > t0; hi -= kBpRows) {
        const int lo = max(hi - kBpRows, t0);
        for (int t = lo + wave; t < hi; t += kBpWaves) {
            const size_t row = (size_t)b * T + t;
            const float* wt = w + row * C * C;
            const int y = min(lane + 1, C - 1);                 // this lane's state (the start state: lane 0 too)
            const float s0 = __int_as_float(bp[row * C]), sy = __int_as_float(bp[row * C + y]);
            const float wb = wt[(size_t)y * C], w00 = wt[0];
            // (what is no number, an arc out of a state that no path is in, is no candidate: the chain's maxima pass over it)
            const float x0 = __fadd_rn(s0, wt[y]);
            const bool any = x0 > LAST_NEG_INF;
            float best = any ? x0 : LAST_NEG_INF;
            int src = any ? 0 : -1;
            constexpr int UN = 8;
            for (int k0 = 1; k0 < C; k0 += UN) {
                float v[UN];
#pragma unroll
                for (int u = 0; u < UN; ++u) v[u] = wt[(size_t)min(k0 + u, C - 1) * C + y];
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int k = k0 + u;
                    const float sk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sy), min(k, C - 1) - 1));
                    const float x = __fadd_rn(sk, v[u]);
                    const bool up = k < C && x > best;          // (ascending states: the first maximum stays)
                    best = up ? x : best;
                    src = up ? k : src;
                }
            }
            const float xk = __fadd_rn(sy, wb), xb = xk > LAST_NEG_INF ? xk : LAST_NEG_INF, xs = __fadd_rn(s0, w00);
            const int fl = best == LAST_NEG_INF ? 0x7fffffff : src * C + y, fb = xb == LAST_NEG_INF ? 0x7fffffff : y * C;
            const bool label = best > xb || (best == xb && fl < fb);
            const int flat = label ? fl : fb, arc = flat == 0x7fffffff ? -1 : flat;
            if (lane + 1 < C) {
                bp[row * C + y] = arc;
                prev[t - lo][y] = (unsigned char)bt_prev_state(arc, C, C);
            }
            if (lane == 0) {
                bp[row * C] = xs > LAST_NEG_INF ? 0 : -1;
                prev[t - lo][0] = 0;
            }
        }
        __syncthreads();
        if (tid < C)
            for (int t = hi - 1; t >= lo; --t) q = prev[t - lo][q];
        __syncthreads();
    }
    if (tid < C) map[((size_t)b * nseg + seg) * C + tid] = q;
}

}  // namespace last
