// Full 2-gram contexts with dense weights: the recursions of Eq. 2 (arXiv
// 2304.13134) in both directions and the tropical one (Section 4.2.3), each
// item and direction on a cluster of K workgroups of one XCD.
//
// With the states written as q = a V + b (b the last label 1..V, a the label
// before it, a = 0 for a history of one label, q = 0 the empty history) the
// label arcs out of the V+1 states with last label b lead to b V + y and
// nowhere else.  Workgroup k owns nb last labels, i.e. for every a a
// contiguous run of nb rows (nb (V+1) floats) of each frame:
//   forward : new[b V + y] = (+)_a cur[a V + b] w[a V + b][y] needs own rows only;
//   backward: new[a V + b] = (+)_y w[a V + b][y] nxt[b V + y] likewise;
// and the V x V transpose between "produced for (b, y)" and "owned by y" is
// the one exchange per frame, through the XCD's L2 (tagged 64-bit words, see
// cluster_kernels.hpp).  The empty label keeps the state and needs none.
//
// Everything is in the log domain (natural logarithms, float32 relative to a float64
// offset per frame, the offset being the largest entry of the frame), so there is no limit on
// the dynamic range of the weights, and scores are rounded as in solo_kernels.hpp (in
// base 2 they would be 1.44 times larger, and so would their roundings).  The tropical recursion adds float32 scores
// and keeps (score, source) exactly as solo_viterbi does.
//
// What bounds it: the chain of a frame.  Own rows -> partial sums (compute
// waves) -> barrier -> combine and publish (exchange waves) -> L2 round trip
// -> own states -> barrier; a wave issues an instruction every five clocks or so, so that what is on this chain counts by
// instructions.  In the log semiring (up to 43 labels) the compute waves therefore form e^w / 4^k of the next frame while the
// exchange is under way, 4^k next to the largest e^w of a thread's rows in a column (backward: of a row), and the exchange waves keep the
// exponentials of the states beside the states: the sums are multiply-adds, the exchange waves have what the partial sums are
// to be multiplied by before these are there, and rows are stored behind the barrier.  A sum that comes out below 2^-92 (weights or
// states far apart) is taken again from the logarithms by the wave that has it, so there is still no limit on the range.
// Weights are requested four rows' worth at a time with
// 16-byte loads two frames (backward: up to four) ahead by waves that never wait
// for an exchange; the exchange waves issue no weight loads, because a wave's
// loads return in order and a look at the exchange would queue behind them.
// Forward and backward pass run at the same time on different compute units.
// Arc marginals are formed afterwards from the stored state vectors by
// dense_marginals_kernel, which streams at memory speed on the whole chip;
// forming them inside the recursion would put the stores on the chain to save
// 4 of 16 bytes per arc.
//
// Measured: 8 items, 200 to 300 frames, 32 labels, loss with gradient 0.61 ms (0.70 with exponentials on the chain) against
// 34 ms with one workgroup per item (solo_kernels.hpp), 1.6 us a frame (1.8) and
// marginals in 0.11 ms; distance of 4 items, 1000 frames, 64 labels (weights in memory) 1.6 ms on 32 workgroups a direction,
// 2.1 on 16 that own twice the labels; 6 items, 120 to 250 frames, 28 labels, shortest path 0.38
// against 3.7 ms.
// What made the difference between 3.0 and 1.9 us a frame, before that, is that every weight
// request and store is issued on every path (the waits for the weights can then
// be counted; a condition around one of them turns them into waits for all) and
// that the exchange waves read all partial results in one batch.
#pragma once
#include "cluster_kernels.hpp"
#include "common.hpp"
#include "numerator_kernels.hpp"
#include "solo_kernels.hpp"

namespace last {

struct TriArgs {
    const float* w;
    const int* len;
    float* alpha;        // log: rows of C floats (natural logs); tropical: final scores [B][C]
    float* beta;
    double* offa;        // offsets of the rows
    double* offb;
    int* bp;             // tropical: [B][T][C] flat arc indices (may be null)
    u64* x;              // exchange slots [clusters][roles][2][xs]
    int* fail;           // [B] set when a workgroup gave up waiting
    int B, T, V, C;
    int nb, K, ncl, G, xs;
    int roles;           // 2: forward and backward, 1: forward only
    int across;          // 1: the directions of an item on two XCDs
    int keep;            // 1: every row is stored at [b][T+1][C]; 0: only the meeting row at [b][C]
    int spin_limit;
};

// row of the state vectors at which the two directions are joined into the distance
__host__ __device__ inline int tri_meet(int L, bool keep) { return keep ? L : (L + 1) / 2; }

constexpr int kTriMaxV = 64;
constexpr int kTriPad = 72;      // floats behind the tile that a row's lanes may read
constexpr int kTriMaxG = 12;     // row groups whose partial results the exchange waves combine

// NW waves of which NCM exchange and the rest compute, nb V <= 64 NCM; NR: 16-byte pieces of a frame per
// compute thread; EPL: elements of a row per lane in the backward direction (four lanes a row, two rows a lane)
template <int NW_, int NCM_, int NR_, int EPL_, bool AHEAD_ = (NR_ <= 4)>
struct TriDims {
    static constexpr int NW = NW_, NCM = NCM_, NR = NR_, EPL = EPL_;
    static constexpr int CT = (NW - NCM) * kWave;              // compute threads
    static constexpr int NP = 2;
    static constexpr int MaxV = 4 * EPL - 1 < kTriMaxV ? 4 * EPL - 1 : kTriMaxV;
    static constexpr int States = NCM * kWave + 32;            // own states, the start state
    static constexpr int BtPitch = (4 * EPL) | 1;              // odd: neighbouring labels start in other banks
    static constexpr int Pitch = NCM * kWave + 32;             // forward, partial results of a row group: 4 CQ floats at most
    // log: the exponentials of the weights are formed beside the exchange.  Not beyond 43 labels, where their registers are
    // not there (64 labels 3.1 -> 4.2 us a frame, spilled), nor in a single workgroup, which has no exchange (8 labels 118 -> 133 us
    // for 100 frames); at 32 labels 1.84 -> 1.47 us a frame
    static constexpr bool Ahead = AHEAD_;
};

constexpr float kLn2 = 0.6931471805599453f;

// log of a sum of e^x from the largest x and the sum of e^(x - m); -inf for m = -inf
__device__ __forceinline__ float ln_sum(float m, float z)
{
    return m == LAST_NEG_INF ? LAST_NEG_INF : fmaf(__builtin_amdgcn_logf(z), kLn2, m);
}
__device__ __forceinline__ float tri_exp(float d) { return fast_exp2(d * kLog2e); }
// e^d for d <= 0 that is good to the hardware's exp2 however large d is: what the product with log2 e is rounded by goes with it.
// Below -150 it is 0 (the remainder of -inf would be none); NaN stays NaN.
__device__ __forceinline__ float tri_exp_far(float d)
{
    d = __builtin_elementwise_maximum(d, -150.f);
    const float p = d * kLog2e, e = fast_exp2(p);
    return fmaf(e, fmaf(-p, kLn2, d), e);
}
// Where the exponentials of weights are formed before their sums, the reference of a set of weights is a power of four next to
// its largest one, m: w log2 e - 2k is rounded once, and k and the exponent of a sum are added up exactly before they meet its
// logarithm.  Relative to the largest weight itself a marginal's error was 1.1 to 1.6 times that of the sums of e^(x - m) (weights of
// 3 to 10 standard deviations; now 0.87 to 1.03 times).  Weights of kTriLarge and more (masks of -1e9, lowest values), where k has no
// place for that, are taken relative to m, and k stands for it to a unit of its last place, which is one of the score.
constexpr float kTriLarge = 5.0e6f;
constexpr float kTriLeast = -3.402823e38f;
constexpr float kTriNone = -1.0e8f;                     // below every 2k of weights that are not large
constexpr float kTriLog2eLow = 1.925963033500e-8f;      // log2 e - (float)log2 e
constexpr float kLn4Down = 1.38629424571990966796875f, kLn4Rest = 1.1540000e-7f;      // log 4 from below, so that -inf stays -inf
// k; -inf where there is no weight.  (Powers of four, so that lowest values have one.)
__device__ __forceinline__ float tri_ref(float m) { return ceilf(m * (0.5f * kLog2e)); }
__device__ __forceinline__ float tri_ref_large(float m) { return m == LAST_NEG_INF ? m : tri_ref(fmaxf(m, kTriLeast)); }
// below kTriInfBits where m is large: |m| - kTriLarge is between 0 and infinity
__device__ __forceinline__ unsigned tri_large(float m) { return __float_as_uint(fabsf(m) - kTriLarge); }
constexpr unsigned kTriInfBits = 0x7f800000u;
// 2k for tri_factor
__device__ __forceinline__ float tri_down(float k) { return fmaxf(k + k, kTriNone); }
// e^w 2^-down; 0 for -inf, also where there is no weight
__device__ __forceinline__ float tri_factor(float w, float down)
{
    return fast_exp2(fmaf(w, kTriLog2eLow, fmaf(w, kLog2e, -down)));
}
// log(4^k z)
__device__ __forceinline__ float tri_ln(float k, float z)
{
    const float n = fmaf((float)__builtin_amdgcn_frexp_expf(z), 0.5f, k);
    return fmaf(n, kLn4Down, fmaf(__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(z)), kLn2, n * kLn4Rest));
}
__device__ __forceinline__ float tri_lse2(float x, float y)     // log(e^x + e^y)
{
    const float m = fmaxf(x, y), lo = fminf(x, y);
    const float d = m == LAST_NEG_INF ? 0.f : lo - m;
    return fmaf(__builtin_amdgcn_logf(1.f + tri_exp(d)), kLn2, m);
}

__device__ __forceinline__ float4 tri_load4(buf_t r, unsigned voff, unsigned soff)      // 4-byte aligned
{
    typedef decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0)) b128_t;
    return __builtin_bit_cast(float4, (b128_t)__builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

template <int CTRL>
__device__ __forceinline__ float tri_quad(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float tri_quad_max(float v)
{
    v = fmaxf(v, tri_quad<0xB1>(v));     // lanes 1,0,3,2
    return fmaxf(v, tri_quad<0x4E>(v));  // lanes 2,3,0,1
}
__device__ __forceinline__ float tri_quad_sum(float v)
{
    v += tri_quad<0xB1>(v);
    return v + tri_quad<0x4E>(v);
}

// largest float of the wave, the same in all lanes, in as few instructions as it takes
__device__ __forceinline__ float tri_wave_max(float v)
{
    asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 0"
        : "+v"(v));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// One look after the other at this lane's word (and, with HEAD, at one header word) until the tags are
// right in every lane of the wave; false when the bound is reached.  The tropical waves look right after they have
// published: in clusters of more than four workgroups (`later`) a first look that leaves 256 clocks later is answered when there
// is something to see, one that leaves at once has to be sent again.  Paths of 200 frames, 1 and 4 items, without and with the delay:
// 22 labels on 5 workgroups 291 / 274 us, 28 labels on 7 304 / 287; but 16 labels on 2, 100 frames, 132 / 139.  The others
// form their header word meanwhile, and are slower for any such wait (1.47 -> 1.60 us a frame).  With two looks under
// way both are slower; so are later looks without the pause between them (28 labels 287 -> 289).
template <bool HEAD, bool TAG16>
__device__ __forceinline__ bool tri_poll(const u64* wp, const u64* hp, bool act, unsigned tag, int limit,
                                         u64& word, u64& head, bool later = false)
{
    if (TAG16 && later) __builtin_amdgcn_s_sleep(4);
    for (int n = 0; n <= limit; ++n) {
        word = xload(wp);
        if (HEAD) head = xload(hp);
        bool ok = TAG16 ? (unsigned)(word >> 48) == (tag & 0xffffu) : (unsigned)(word >> 32) == tag;
        ok = ok || !act;
        if (HEAD) ok = ok && (unsigned)(head >> 32) == tag;
        if (__all(ok)) return true;
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// A lane's place in an exchange slot as a byte offset in a register of its own: the scalar registers are all taken, and an
// address put together from uniform parts that were put away costs their reads from a vector register's lanes
// on the chain of every frame.
__device__ __forceinline__ unsigned tri_place(int word)
{
    unsigned off = 8u * (unsigned)word;
    asm volatile("" : "+v"(off));
    return off;
}
__device__ __forceinline__ u64* tri_at(u64* slot, unsigned off) { return (u64*)((char*)slot + off); }

// what the two directions share: which part of the lattice a workgroup owns, and its pieces of a frame
struct TriOwn {
    int V, V1, k, b0, nbk;       // own last labels b0 .. b0 + nbk - 1
    int W, CQ, G;                // floats and 16-byte pieces of a row run, row groups
    int rows;                    // own states with at least one label: (V + 1) nbk
};

// static LDS of either direction
template <typename D>
struct TriLds {
    float own[D::States + 32];                 // own states, [a nbk + i]; the start state at [rows]; then nbk times -inf
    float ex[D::States + 32];                  // log: their exponentials
    float bl[D::States];                       // tropical: empty-label candidates; backward: the new states
    float bw[2][D::States + 32];               // forward, log: weights of the empty label
    int far[2];                                // log: a sum of the frame was taken the long way
    float strow[2][4 * 17 + 4];                // the start state's row of weights
    float xl[D::NCM * kWave + kTriMaxV];       // exchange of a single workgroup (K = 1)
    int xa[D::NCM * kWave];
    int flat[D::States];                       // tropical: backpointers of the frame
    double off;                                // offset of the own states
    float hd[8];
    int dead;
};

// a lane that must not store gets an offset outside the descriptor; every store is issued on every path, so that
// the waits for prefetched weights can be counted
constexpr unsigned kTriOut = 0xfffffff0u;

// A sum of products e^x e^(w - m), both factors at most 1, is the sum it stands for as long as it is not below this: what both
// factors have lost below 2^-126 is 2^-30 of it at most.  Smaller ones (weights far apart, states out of reach) are
// taken from the logarithms themselves.  A sum of states that no path is in is -0, which stands for itself: their exponentials are -0;
// its weights are no reference for the sums of others.
constexpr float kTriFar = 2.0194839e-28f;      // 2^-92
// A wave that had one takes the logarithms at once for the next kTriSkip - 1 frames.  Against sums of differences in all frames, 100
// frames of one item and 60 of eight, without / with that: normal weights, 12 to 40 labels 0.84 to 0.94 / 0.85 to 0.97 of the time,
// 20 standard deviations 1.07 to 1.29 / 1.04 to 1.17, a label at -1e9 0.98 to 1.12 / 0.95 to 1.08, half of the arcs missing 0.90 to
// 1.11 / 0.88 to 1.07.
constexpr int kTriSkip = 16;

template <typename D, bool TROP>
__device__ __forceinline__ void tri_forward(const TriArgs& a, const TriOwn& o, int b, int L, unsigned& gstep,
                                            u64* xbase, TriLds<D>& s, float* dyn)
{
    constexpr int NCM = D::NCM;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));     // (what one direction derives from it is not kept in registers through the other)
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool comm = wave < NCM;
    const int V = o.V, V1 = o.V1, nbk = o.nbk;
    constexpr bool AHEAD = !TROP && D::Ahead;
    const int P = AHEAD ? D::Pitch : 4 * o.CQ;
    float* ps = dyn;                            // [kTriMaxG][P] partial sums   (tropical: source a, as int)
    float* pm = dyn + kTriMaxG * P;             // [kTriMaxG][P] partial maxima (tropical: scores); log: two frames of them
    const int pmz = AHEAD ? kTriMaxG * P : 0;
    const size_t fr = (size_t)o.V1 * a.C;
    const float* wi = a.w + (size_t)b * a.T * fr;
    const int steps = TROP || a.keep ? L : tri_meet(L, false);

    for (int r = tid; r < D::States + 32; r += D::NW * kWave) {
        s.own[r] = r == o.rows ? 0.f : LAST_NEG_INF;
        if (AHEAD) s.ex[r] = r == o.rows ? 1.f : -0.f;
    }
    for (int i = tid; i < kTriMaxG * P; i += D::NW * kWave) {      // groups that do not exist stay neutral
        pm[i] = LAST_NEG_INF;
        if (AHEAD) pm[pmz + i] = LAST_NEG_INF;
        ps[i] = TROP ? __int_as_float(0xffff) : AHEAD ? -0.f : 0.f;
    }
    if (tid == 0) { s.dead = 0; s.off = 0.0; s.far[0] = s.far[1] = 0; }
    __syncthreads();

    if (!comm) {
        const int ct = tid - NCM * kWave;
        const int g = ct / o.CQ, cq = ct - g * o.CQ;
        const bool act = g < o.G;
        const int gc = act ? g : 0;
        const int col0 = min(4 * cq, o.W - 4);
        int iC[4], cB = 0, iB = 0;
        bool hasB = false;                                     // one of the four columns is an empty label's (V >= 3)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            iC[c] = (col0 + c) / V1;
            if (act && col0 + c == iC[c] * V1) { hasB = true; cB = c; iB = iC[c]; }
        }
        // pieces n = 0 .. nl - 1 of a thread are rows g + G n of every frame, piece nl may be past the last row
        // (its states then read -inf), pieces beyond nl repeat it
        const int nl = V / o.G, rl = gc + o.G * nl;
        const unsigned off0 = 4u * (unsigned)((gc * V + o.b0) * V1 + col0), offL = 4u * (unsigned)((min(rl, V) * V + o.b0) * V1 + col0);
        const unsigned stoff = 4u * (unsigned)min(lane, V), frb = 4u * (unsigned)fr;
        const int dOff = 4 * o.G * V * V1;
        const int base0 = gc * nbk, dBase = o.G * nbk, baseN = o.rows + 1;
        const int baseL = rl <= V ? rl * nbk : baseN;
        auto base = [&](int n) __attribute__((always_inline)) { return n < nl ? base0 + n * dBase : n == nl ? baseL : baseN; };
        // own states -> a row in memory: compute thread <-> own state, the start state from the first workgroup
        const bool rok = ct < o.rows || (ct == o.rows && o.k == 0);
        const int rS = min(ct, o.rows);
        const unsigned rq = rok ? 4u * (unsigned)(ct < o.rows ? (ct / nbk) * V + o.b0 + ct % nbk : 0) : kTriOut;
        const unsigned oq = ct == 0 && o.k == 0 ? 0u : kTriOut;
        const unsigned rowb = (unsigned)a.C * 4u;
        auto store_row = [&](int t, bool on) __attribute__((always_inline)) {
            const size_t row = !TROP && a.keep ? (size_t)b * (a.T + 1) + t : (size_t)b;
            buf_store(s.own[rS], make_buf(a.alpha + row * a.C, on ? rowb : 0u), rq, 0);
            if (!TROP) nw_store64(s.off, make_buf(a.offa + row, on ? 8u : 0u), oq, 0);
        };
        // the same in two: read before the exchange, stored beside it
        auto store_read = [&](float x, double at, int t) __attribute__((always_inline)) {
            const size_t row = a.keep ? (size_t)b * (a.T + 1) + t : (size_t)b;
            buf_store(x, make_buf(a.alpha + row * a.C, a.keep ? rowb : 0u), rq, 0);
            nw_store64(at, make_buf(a.offa + row, a.keep ? 8u : 0u), oq, 0);
        };
        float4 wv[2][D::NR];
        float st[2] = {0.f, 0.f}, st64[2] = {0.f, 0.f};
        auto issue = [&](auto S, int t) __attribute__((always_inline)) {
            const buf_t rs = make_buf(wi + (size_t)min(t, L - 1) * fr, frb);
#pragma unroll
            for (int n = 0; n < D::NR; ++n)
                wv[decltype(S)::value][n] = tri_load4(rs, n < nl ? off0 : offL, (unsigned)(n < nl ? n * dOff : 0));
            st[decltype(S)::value] = buf_load(rs, stoff, 0);
            if (D::MaxV == 64) st64[decltype(S)::value] = buf_load(rs, 4u * (unsigned)V, 0);
        };
        auto start_row = [&](auto S) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            if (wave == D::NW - 1) {
                if (lane <= V) s.strow[Z][lane] = st[Z];
                if (D::MaxV == 64) s.strow[Z][V] = st64[Z];
            }
        };
        // log: exponentials of a frame's weights relative to the largest of the thread's rows in a column (tri_ref), and what the exchange
        // waves need of it before its sums; ahead of the chain.  z0: negative where a small sum is of no account (a column without a
        // weight, whose reference makes it -0, or of the empty label)
        float E[AHEAD ? D::NR : 1][4], z0[4];
        unsigned exOff[AHEAD ? D::NR : 1][4];
        if constexpr (AHEAD) {
#pragma unroll
            for (int n = 0; n < D::NR; ++n) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    exOff[n][c] = 4u * (unsigned)(base(n) + iC[c]);
                    asm volatile("" : "+v"(exOff[n][c]));           // (an instruction less on the chain)
                }
            }
        }
        auto factors = [&](auto S) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            int at = hasB ? cB : -1;
            asm volatile("" : "+v"(at));                        // (no masks kept in scalar registers for all frames)
            float mw[4] = {LAST_NEG_INF, LAST_NEG_INF, LAST_NEG_INF, LAST_NEG_INF};
#pragma unroll
            for (int n = 0; n < D::NR; ++n) {
                const float4 w4 = wv[Z][n];
                const float wc[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) mw[c] = fmaxf(mw[c], wc[c]);
            }
            // The empty label's weights, at the places of the states that they are added to.  (Through the states' own offsets: with offsets
            // of their own the kernel of up to 35 labels took 113 registers.  One gets eight more than 112, and beside two workgroups of it
            // a SIMD then has no room for a wave of the numerator's gather, beside one for four instead of five: loss on on-the-fly
            // weights, 16 items, 1024 frames, 32 labels, 512 hidden units 11.25 -> 11.12 ms.)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (at == c) {
#pragma unroll
                    for (int n = 0; n < D::NR; ++n) {
                        const float4 w4 = wv[Z][n];
                        *(float*)((char*)s.bw[Z] + exOff[AHEAD ? n : 0][c]) = c == 0 ? w4.x : c == 1 ? w4.y : c == 2 ? w4.z : w4.w;
                    }
                }
            unsigned large = ~0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) large = min(large, tri_large(mw[c]));
            const bool any_large = __any(large < kTriInfBits);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float m = mw[c];
                float down;
                if (__builtin_expect(any_large, 0)) {
                    const bool go = tri_large(m) < kTriInfBits;
                    mw[c] = tri_ref_large(m);
                    down = go ? 0.f : tri_down(mw[c]);
#pragma unroll
                    for (int n = 0; n < D::NR; ++n) {
                        const float4 w4 = wv[Z][n];
                        const float wc = c == 0 ? w4.x : c == 1 ? w4.y : c == 2 ? w4.z : w4.w;
                        E[AHEAD ? n : 0][c] = tri_factor(go ? wc - m : wc, down);
                    }
                } else {
                    mw[c] = tri_ref(m);
                    down = tri_down(mw[c]);
#pragma unroll
                    for (int n = 0; n < D::NR; ++n) {
                        const float4 w4 = wv[Z][n];
                        const float wc = c == 0 ? w4.x : c == 1 ? w4.y : c == 2 ? w4.z : w4.w;
                        E[AHEAD ? n : 0][c] = tri_factor(wc, down);
                    }
                }
                z0[c] = m == LAST_NEG_INF || c == at ? -1.0e30f : -0.f;
            }
            if (act) *(float4*)(pm + Z * pmz + g * P + 4 * cq) = make_float4(mw[0], mw[1], mw[2], mw[3]);
        };
        if (steps > 0) {
            issue(std::integral_constant<int, 0>(), 0);
            issue(std::integral_constant<int, 1>(), 1);
            start_row(std::integral_constant<int, 0>());
            if constexpr (AHEAD) factors(std::integral_constant<int, 0>());
        }
        __syncthreads();
        int skip = 0;                            // log: frames to take the long way, see kTriSkip
        auto frame = [&](auto S, int t) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            float rowv = 0.f;
            double rowo = 0.0;
            if (TROP) {
                if (t > 0) buf_store(__int_as_float(s.flat[rS]), make_buf(a.bp + ((size_t)b * a.T + t - 1) * a.C, a.bp ? rowb : 0u), rq, 0);
            } else if (!AHEAD) {
                store_row(t, a.keep);
            }
            bool far = true;
            if constexpr (AHEAD) {
                rowv = s.own[rS];
                rowo = s.off;
                skip = __builtin_amdgcn_readfirstlane(skip) - 1;
            }
            if (AHEAD && __builtin_expect(skip < 0, 1)) {
                float z[4] = {z0[0], z0[1], z0[2], z0[3]};
                float x[D::NR][4];
#pragma unroll
                for (int n = 0; n < D::NR; ++n)
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[n][c] = *(const float*)((const char*)s.ex + exOff[AHEAD ? n : 0][c]);
#pragma unroll
                for (int n = 0; n < D::NR; ++n)
#pragma unroll
                    for (int c = 0; c < 4; ++c) z[c] = fmaf(x[n][c], E[AHEAD ? n : 0][c], z[c]);
                const unsigned least = min(min(min(__float_as_uint(z[0]), __float_as_uint(z[1])), __float_as_uint(z[2])), __float_as_uint(z[3]));
                far = __any(least < __builtin_bit_cast(unsigned, kTriFar));
                skip = far ? kTriSkip : 0;
                if (act) *(float4*)(ps + g * P + 4 * cq) = make_float4(z[0], z[1], z[2], z[3]);
            }
            if (__builtin_expect(far, !AHEAD)) {
            float m[4], z[4];
            int src[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { m[c] = LAST_NEG_INF; z[c] = 0.f; src[c] = 0xffff; }
            // at most three rows at a time (registers)
#pragma unroll
            for (int n0 = 0; n0 < D::NR; n0 += 3) {
                constexpr int N3 = D::NR < 3 ? D::NR : 3;
                float q[N3][4], mo[4];
#pragma unroll
                for (int n = 0; n < N3; ++n)
                    if (n0 + n < D::NR) {
                        const int bs = base(n0 + n);
#pragma unroll
                        for (int c = 0; c < 4; ++c) q[n][c] = s.own[bs + iC[c]];
                    }
#pragma unroll
                for (int c = 0; c < 4; ++c) mo[c] = m[c];
#pragma unroll
                for (int n = 0; n < N3; ++n) {
                    if (n0 + n >= D::NR) continue;
                    const float4 w4 = wv[Z][n0 + n];
                    const float wc[4] = {w4.x, w4.y, w4.z, w4.w};
                    float xB = LAST_NEG_INF;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x = __fadd_rn(q[n][c], wc[c]);
                        q[n][c] = x;
                        xB = c == cB ? x : xB;
                        if (TROP) {
                            const bool up = x > m[c];          // (ascending a: the first maximum stays)
                            m[c] = up ? x : m[c];
                            src[c] = up ? gc + o.G * (n0 + n) : src[c];
                        } else {
                            m[c] = fmaxf(m[c], x);
                        }
                    }
                    const int bs = base(n0 + n);
                    if (!AHEAD && hasB && bs <= o.rows) s.bl[bs + iB] = xB;
                }
                if (!TROP) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float mm = m[c] == LAST_NEG_INF ? 0.f : m[c];
                        if (n0 > 0) z[c] *= tri_exp(mo[c] - mm);
#pragma unroll
                        for (int n = 0; n < N3; ++n)
                            if (n0 + n < D::NR) z[c] += tri_exp(q[n][c] - mm);
                    }
                }
            }
            if (AHEAD) {
                // the sums relative to the reference
                unsigned large = ~0u;
#pragma unroll
                for (int c = 0; c < 4; ++c) large = min(large, tri_large(m[c]));
                if (__builtin_expect(__any(large < kTriInfBits), 0)) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float k = tri_ref_large(m[c]);
                        z[c] *= tri_large(m[c]) < kTriInfBits ? 1.f : tri_factor(m[c], tri_down(k));
                        m[c] = k;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float k = tri_ref(m[c]);
                        z[c] *= tri_factor(m[c], tri_down(k));
                        m[c] = k;
                    }
                }
            }
            if (act) {
                *(float4*)(pm + Z * pmz + g * P + 4 * cq) = make_float4(m[0], m[1], m[2], m[3]);
                if (TROP) *(int4*)(ps + g * P + 4 * cq) = make_int4(src[0], src[1], src[2], src[3]);
                else *(float4*)(ps + g * P + 4 * cq) = make_float4(z[0], z[1], z[2], z[3]);
            }
            if (AHEAD) s.far[Z] = 1;
            }
            lds_only_barrier();                                                   // B
            if (a.K == 1) lds_only_barrier();
            // (the exchange is under way) start row of the next frame, weights of the frame after it
            start_row(std::integral_constant<int, Z ^ 1>());
            issue(S, t + 2);
            if constexpr (AHEAD) {
                store_read(rowv, rowo, t);
                factors(std::integral_constant<int, Z ^ 1>());
            }
            lds_only_barrier();                                                   // A
        };
        for (int t = 0; t < steps; t += 2) {
            frame(std::integral_constant<int, 0>(), t);
            if (t + 1 < steps) frame(std::integral_constant<int, 1>(), t + 1);
        }
        store_row(steps, true);
        if (TROP && steps > 0)
            buf_store(__int_as_float(s.flat[rS]), make_buf(a.bp + ((size_t)b * a.T + steps - 1) * a.C, a.bp ? rowb : 0u), rq, 0);
    } else {
        // published state (b0 + i, y) of this lane and the word of its own state (ga, b0 + gi)
        const int lidx = wave * kWave + lane;
        const bool act = lidx < nbk * V;
        const int pi = act ? lidx / V : 0, py = act ? lidx - pi * V + 1 : 1;
        const int col = pi * V1 + py;
        const int slot = col + (col >= 4 * (o.CQ - 1) ? 4 * o.CQ - o.W : 0);
        const int ga = act ? lidx / nbk + 1 : 1, gi = act ? lidx - (ga - 1) * nbk : 0;
        const int grow = ga * nbk + gi;                                           // own row of the gathered state
        const int gidx = (ga - 1) * V + (o.b0 - 1 + gi);
        const bool second = wave == 0 && lane <= nbk;                             // histories of one label, the start state
        const bool single = wave == 0 && lane < nbk;
        const int nh = a.K * NCM;
        const unsigned oMine = tri_place((o.b0 - 1) * V + lidx), oGot = tri_place(gidx);
        const unsigned oHead = tri_place(V * V + V + o.k * NCM + wave), oHeads = tri_place(V * V + V + (lane < nh ? lane : 0));
        bool dead = false;
        double A = 0.0;
        float mine = LAST_NEG_INF, mine1 = LAST_NEG_INF;        // log: own states of this lane (the gathered one; with one label)
        __syncthreads();
        for (int t = 0; t < steps; ++t) {
            u64* xs = xbase + (size_t)(gstep & 1) * a.xs;
            const unsigned tag = gstep + 1;
            gstep += 1;
            // log: what the partial sums will have to be multiplied by, while they are formed
            float fz[AHEAD ? kTriMaxG : 1], top = LAST_NEG_INF;
            auto scales = [&](auto&& counts) __attribute__((always_inline)) {
                const float* r = pm + (t & 1) * pmz + slot;
                top = LAST_NEG_INF;
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) fz[AHEAD ? g : 0] = counts(r[g * P], g);
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) top = fmaxf(top, fz[AHEAD ? g : 0]);
                const float mm = fmaxf(top, kTriLeast);
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) {
                    const float d = fz[AHEAD ? g : 0] - mm;
                    fz[AHEAD ? g : 0] = fast_exp2(d + d);
                }
            };
            auto all = [](float k, int) __attribute__((always_inline)) { return k; };
            if constexpr (AHEAD) {
                scales(all);
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) asm volatile("" : "+v"(fz[g]));        // (not put off behind the barrier)
                asm volatile("" : "+v"(top));
            }
            float bwr = LAST_NEG_INF, u2 = LAST_NEG_INF;       // the empty label's candidate; histories of one label, the start state
            if constexpr (AHEAD) {
                bwr = act ? mine + s.bw[t & 1][grow] : LAST_NEG_INF;
                const float w0 = s.strow[t & 1][single ? o.b0 + lane : 0], start = s.own[o.rows], kept = mine1 + s.bw[t & 1][single ? lane : 0];
                u2 = tri_lse2(second ? __fadd_rn(start, w0) : LAST_NEG_INF, single ? kept : LAST_NEG_INF);
                asm volatile("" : "+v"(bwr), "+v"(u2));
            }
            lds_only_barrier();                                                   // B
            float val = LAST_NEG_INF, m[kTriMaxG], z[kTriMaxG];
            int src = 0xffff;
            if (!AHEAD) {
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) m[g] = pm[g * P + slot];
            }
#pragma unroll
            for (int g = 0; g < kTriMaxG; ++g) z[g] = ps[g * P + slot];
            const int far = AHEAD ? s.far[t & 1] : 0;
            const float blr = AHEAD ? bwr : s.bl[grow];
            const float w0 = AHEAD ? 0.f : s.strow[t & 1][single ? o.b0 + lane : 0], start = AHEAD ? 0.f : s.own[o.rows], sbr = AHEAD ? 0.f : s.bl[single ? lane : 0];
            if (!AHEAD) {
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) val = fmaxf(val, m[g]);
            }
            if (TROP) {
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) src = min(src, m[g] == val ? __float_as_int(z[g]) : 0xffff);
                if (val == LAST_NEG_INF) src = 0xffff;
            } else if (!AHEAD) {
                const float mm = val == LAST_NEG_INF ? 0.f : val;
                float zz = 0.f;
#pragma unroll
                for (int g = 0; g < kTriMaxG; ++g) zz += z[g] * tri_exp(m[g] - mm);
                val = ln_sum(val, zz);
            } else {
                if (__builtin_expect(__builtin_amdgcn_readfirstlane(far), 0)) {
                    scales(all);
                }
                auto total = [&]() __attribute__((always_inline)) {
                    float zz = -0.f, zy = -0.f;
#pragma unroll
                    for (int g = 0; g < kTriMaxG; g += 2) {
                        zz = fmaf(z[g], fz[AHEAD ? g : 0], zz);
                        zy = fmaf(z[g + 1], fz[AHEAD ? g + 1 : 0], zy);
                    }
                    return zz + zy;
                };
                float sum = total();
                // The group with the largest weights may have no state that a path is in, and the others may then be nothing beside them.
                // (-0: there is no such state at all.)
                if (__builtin_expect(__any(__float_as_uint(sum) < __builtin_bit_cast(unsigned, kTriFar)), 0)) {
                    scales([&](float k, int g) __attribute__((always_inline)) { return z[g] <= 0.f ? LAST_NEG_INF : k; });
                    sum = total();
                }
                val = tri_ln(top, sum);
            }
            const float blg = AHEAD || act ? blr : LAST_NEG_INF;
            // histories of one label: from the start state, or kept by the empty label; the start state: kept
            const float sn = AHEAD || !second ? LAST_NEG_INF : __fadd_rn(start, w0);
            const float sb = !AHEAD && single ? sbr : LAST_NEG_INF;
            float head = LAST_NEG_INF;
            u64 word = 0, hw = 0;
            if (a.K == 1) {
                if (!TROP) head = tri_wave_max(fmaxf(fmaxf(act ? val : LAST_NEG_INF, blg), AHEAD ? u2 : fmaxf(sn, sb)));
                if (act) { s.xl[lidx] = val; s.xa[lidx] = src; }
                if (lane == 0) s.hd[wave] = head;
                lds_only_barrier();
                const int wl = (ga - 1) * V + gi;                                 // (b0 = 1)
                val = s.xl[act ? wl : 0];
                src = s.xa[act ? wl : 0];
                head = s.hd[lane < NCM ? lane : 0];
            } else {
                if (act) xpublish(tri_at(xs, oMine), TROP ? (u64)__float_as_uint(val) | ((u64)(unsigned)src << 32) | ((u64)(tag & 0xffffu) << 48)
                                             : pack_word(val, tag));
                if (!TROP) {
                    head = tri_wave_max(fmaxf(fmaxf(act ? val : LAST_NEG_INF, blg), AHEAD ? u2 : fmaxf(sn, sb)));
                    if (lane == 0) xpublish(tri_at(xs, oHead), pack_word(head, tag));
                }
                if (!dead) dead = !tri_poll<!TROP, TROP>(tri_at(xs, oGot), tri_at(xs, oHeads), act, tag, a.spin_limit, word, hw, a.K > 4);
                val = __uint_as_float((unsigned)word);
                src = (int)((word >> 32) & 0xffffu);
                head = __uint_as_float((unsigned)hw);
            }
            if (TROP) {
                // the label candidate against the empty label: higher score, then lower arc
                auto keep = [&](float x, int fx, float y, int fy, int row) __attribute__((always_inline)) {
                    if (x == LAST_NEG_INF) fx = 0x7fffffff;
                    if (y == LAST_NEG_INF) fy = 0x7fffffff;
                    const bool first = x > y || (x == y && fx < fy);
                    const int flat = first ? fx : fy;
                    s.own[row] = first ? x : y;
                    s.flat[row] = flat == 0x7fffffff ? -1 : flat;
                };
                if (act) {
                    const int q = ga * V + o.b0 + gi;
                    keep(dead ? LAST_NEG_INF : val, (src * V + ga) * V1 + o.b0 + gi, blg, q * V1, grow);
                }
                if (single) keep(sn, o.b0 + lane, sb, (o.b0 + lane) * V1, lane);
                if (second && !single) keep(sn, 0, LAST_NEG_INF, 0, o.rows);
            } else {
                float mx = tri_wave_max(head);
                if (mx == LAST_NEG_INF) mx = 0.f;              // no state reachable: keep -inf everywhere
                A += (double)mx;
                if (act) {
                    mine = tri_lse2(val, blg) - mx;
                    if (AHEAD) s.ex[grow] = mine == LAST_NEG_INF ? -0.f : tri_exp_far(mine);
                    s.own[grow] = mine;
                }
                if (second) {
                    mine1 = (AHEAD ? u2 : tri_lse2(sn, sb)) - mx;
                    if (AHEAD) s.ex[single ? lane : o.rows] = mine1 == LAST_NEG_INF ? -0.f : tri_exp_far(mine1);
                    s.own[single ? lane : o.rows] = mine1;
                }
                if (tid == 0) {
                    s.off = A;
                    if (AHEAD) s.far[(t & 1) ^ 1] = 0;
                }
            }
            if (dead) s.dead = 1;
            lds_only_barrier();                                                   // A
        }
    }
    __syncthreads();
    if (tid == 0 && s.dead) a.fail[b] = 1;
    __syncthreads();
}

template <typename D>
__device__ __forceinline__ void tri_backward(const TriArgs& a, const TriOwn& o, int b, int L, unsigned& gstep,
                                             u64* xbase, TriLds<D>& s, float* dyn)
{
    constexpr int NCM = D::NCM;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));     // (what one direction derives from it is not kept in registers through the other)
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool comm = wave < NCM;
    const int V = o.V, V1 = o.V1, nbk = o.nbk, P = 4 * o.CQ;
    constexpr int BP = D::BtPitch;
    constexpr bool AHEAD = D::Ahead;
    const int epl = (V1 + 3) / 4;
    float* bt = dyn;                              // [nbk + 1][BP] states (b0 + i, y) by i; [nbk]: histories of one label
    float* be = dyn + ((a.nb + 1) * BP + 3) / 4 * 4;     // their exponentials
    float* tile = dyn + 2 * (((a.nb + 1) * BP + 3) / 4 * 4);   // [V + 1][P] weights of a frame, two of them
    const int tilez = AHEAD ? V1 * P + kTriPad : 0;
    const size_t fr = (size_t)V1 * a.C;
    const float* wi = a.w + (size_t)b * a.T * fr;
    const int low = a.keep ? 1 : tri_meet(L, false);       // the last row this direction makes
    const int steps = max(L - low, 0);
    const int rows = o.rows + (o.k == 0 ? 1 : 0);          // the first workgroup also has the start state

    for (int r = tid; r <= o.rows; r += D::NW * kWave) {
        s.own[r] = 0.f;
        s.ex[r] = 1.f;
    }
    // (four lanes read at least V + 1 elements of a row; what they read past it counts for nothing)
    for (int i = tid; i < (nbk + 1) * BP; i += D::NW * kWave) {
        bt[i] = i % BP < V1 ? 0.f : LAST_NEG_INF;
        be[i] = i % BP < V1 ? 1.f : 0.f;
    }
    for (int i = tid; i < (AHEAD ? 2 : 1) * (V1 * P + kTriPad); i += D::NW * kWave) tile[i] = 0.f;
    if (tid < 72) s.strow[0][tid] = s.strow[1][tid] = 0.f;
    if (tid == 0) { s.dead = 0; s.off = 0.0; }
    __syncthreads();

    if (!comm) {
        const int ct = tid - NCM * kWave;
        const int g = ct / o.CQ, cq = ct - g * o.CQ;
        const bool act = g < o.G;
        const int gc = act ? g : 0;
        const int col0 = min(4 * cq, o.W - 4);
        const int nl = V / o.G, rl = gc + o.G * nl;             // as in the forward direction
        const unsigned off0 = 4u * (unsigned)((gc * V + o.b0) * V1 + col0), offL = 4u * (unsigned)((min(rl, V) * V + o.b0) * V1 + col0);
        const unsigned stoff = 4u * (unsigned)min(lane, V), frb = 4u * (unsigned)fr;
        const int dOff = 4 * o.G * V * V1;
        const bool rok = ct < o.rows || (ct == o.rows && o.k == 0);
        const int rS = min(ct, o.rows);
        const unsigned rq = rok ? 4u * (unsigned)(ct < o.rows ? (ct / nbk) * V + o.b0 + ct % nbk : 0) : kTriOut;
        const unsigned oq = ct == 0 && o.k == 0 ? 0u : kTriOut;
        const unsigned rowb = (unsigned)a.C * 4u;
        auto store_row = [&](int t, bool on) __attribute__((always_inline)) {
            const size_t row = a.keep ? (size_t)b * (a.T + 1) + t : (size_t)b;
            buf_store(s.own[rS], make_buf(a.beta + row * a.C, on ? rowb : 0u), rq, 0);
            nw_store64(s.off, make_buf(a.offb + row, on ? 8u : 0u), oq, 0);
        };
        float4 wv[2][D::NR];
        float st[2] = {0.f, 0.f}, st64[2] = {0.f, 0.f};
        // step n works on frame L - 1 - n
        auto issue = [&](auto S, int n) __attribute__((always_inline)) {
            const buf_t rs = make_buf(wi + (size_t)max(L - 1 - n, 0) * fr, frb);
#pragma unroll
            for (int x = 0; x < D::NR; ++x)
                wv[decltype(S)::value][x] = tri_load4(rs, x < nl ? off0 : offL, (unsigned)(x < nl ? x * dOff : 0));
            st[decltype(S)::value] = buf_load(rs, stoff, 0);
            if (D::MaxV == 64) st64[decltype(S)::value] = buf_load(rs, 4u * (unsigned)V, 0);
        };
        auto spread = [&](auto S) __attribute__((always_inline)) {                 // registers -> tile
            constexpr int Z = decltype(S)::value;
#pragma unroll
            for (int x = 0; x < D::NR; ++x)
                if (act && g + o.G * x <= V) {
                    float* d = tile + Z * tilez + (g + o.G * x) * P + col0;
                    const float4 v = wv[Z][x];
                    if (col0 & 3) { d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w; }
                    else *(float4*)d = v;
                }
            if (wave == D::NW - 1) {
                if (lane <= V) s.strow[AHEAD ? Z : 0][lane] = st[Z];
                if (D::MaxV == 64) s.strow[AHEAD ? Z : 0][V] = st64[Z];
            }
        };
        // four lanes a row: elements y = l epl .. l epl + epl - 1
        const int l = ct & 3;
        const float* rowP[D::NP];
        const float* btP[D::NP];
        int rP[D::NP], rowZ[D::NP];
#pragma unroll
        for (int p = 0; p < D::NP; ++p) {
            rP[p] = min((ct >> 2) + p * (D::CT / 4), rows - 1);
            const int ra = rP[p] / nbk, ri = rP[p] - ra * nbk;
            rowP[p] = (rP[p] == o.rows ? s.strow[0] : tile + ra * P + ri * V1) + l * epl;
            rowZ[p] = !AHEAD ? 0 : rP[p] == o.rows ? (int)(sizeof(s.strow[0]) / sizeof(float)) : tilez;
            btP[p] = bt + (rP[p] == o.rows ? nbk : ri) * BP + l * epl;
        }
        const int beOff = (int)(be - bt);
        // exponentials of a frame's rows relative to a row's largest weight (tri_ref); ahead of the chain
        // Of the lanes of a row the first takes the logarithm of its first sum, the second that of the other; a sum below `least` is
        // taken the long way.
        float E[AHEAD ? D::NP : 1][D::EPL], least[D::NP], ref = LAST_NEG_INF;
        static_assert(D::NP == 2, "two of the four lanes");
        const int count = max(0, min(epl, V1 - l * epl));       // elements of the row in this lane
        auto factors = [&](auto S) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            int have = count;
            asm volatile("" : "+v"(have));                      // (no masks kept in scalar registers for all frames)
#pragma unroll
            for (int p = 0; p < (AHEAD ? D::NP : 1); ++p) {
                const float* row = rowP[p] + Z * rowZ[p];
                float m = LAST_NEG_INF;
#pragma unroll
                for (int e = 0; e < D::EPL; ++e) {
                    E[p][e] = e < have ? row[e] : LAST_NEG_INF;
                    m = fmaxf(m, E[p][e]);
                }
                m = tri_quad_max(m);
                float k = tri_ref(m), down = tri_down(k);
                if (__builtin_expect(__any(tri_large(m) < kTriInfBits), 0)) {
                    const bool go = tri_large(m) < kTriInfBits;
                    k = tri_ref_large(m);
                    down = go ? 0.f : down;
#pragma unroll
                    for (int e = 0; e < D::EPL; ++e) E[p][e] -= go ? m : 0.f;
                }
                least[p] = k == LAST_NEG_INF ? -1.f : kTriFar;
                ref = p == 0 || l == 1 ? k : ref;
#pragma unroll
                for (int e = 0; e < D::EPL; ++e) E[p][e] = tri_factor(E[p][e], down);
            }
        };
        if (steps > 0) {
            issue(std::integral_constant<int, 0>(), 0);
            issue(std::integral_constant<int, 1>(), 1);
            spread(std::integral_constant<int, 0>());
            issue(std::integral_constant<int, 0>(), 2);
            if (AHEAD) {
                spread(std::integral_constant<int, 1>());
                issue(std::integral_constant<int, 1>(), 3);
            }
        }
        __syncthreads();
        if constexpr (AHEAD)
            if (steps > 0) factors(std::integral_constant<int, 0>());
        int skip = 0;                            // frames to take the long way, see kTriSkip
        auto frame = [&](auto S, int n) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            bool far = true;
            float rowv = 0.f;
            double rowo = 0.0;
            if constexpr (AHEAD) {
                rowv = s.own[rS];
                rowo = s.off;
                skip = __builtin_amdgcn_readfirstlane(skip) - 1;
            }
            if (AHEAD && __builtin_expect(skip < 0, 1)) {
                far = false;
                float sum = 0.f;
#pragma unroll
                for (int p = 0; p < D::NP; ++p) {
                    if (__builtin_amdgcn_readfirstlane(ct >> 2) + p * (D::CT / 4) >= rows) break;      // (no row for this wave)
                    float z = 0.f, z1 = 0.f;
#pragma unroll
                    for (int e = 0; e < D::EPL; ++e) {
                        float x = btP[p][beOff + e];
                        if (e == 0) x = l == 0 ? s.ex[rP[p]] : x;                  // the empty label keeps the state
                        if (e & 1) z1 = fmaf(E[AHEAD ? p : 0][e], x, z1);
                        else z = fmaf(E[AHEAD ? p : 0][e], x, z);
                    }
                    z = tri_quad_sum(z + z1);
                    far = far || !(z >= least[p]);
                    sum = p == 0 || l == 1 ? z : sum;
                }
                const int r = (ct >> 2) + l * (D::CT / 4);
                if (l < D::NP && r < rows) s.bl[r] = tri_ln(ref, sum);
                far = __any(far);
                skip = far ? kTriSkip : 0;
            }
            if (__builtin_expect(far, !AHEAD))
#pragma unroll
            for (int p = 0; p < D::NP; ++p) {
                const int r = (ct >> 2) + p * (D::CT / 4);
                if (r < rows) {
                    const float* row = rowP[p] + Z * rowZ[p];
                    float v[D::EPL], x[D::EPL], m = LAST_NEG_INF;
                    const float keep = s.own[r];                                   // the empty label keeps the state
                    constexpr int EH = D::EPL > 11 ? 9 : D::EPL;                   // (registers)
#pragma unroll
                    for (int e0 = 0; e0 < D::EPL; e0 += EH) {
#pragma unroll
                        for (int e = e0; e < e0 + EH && e < D::EPL; ++e) { x[e] = row[e]; v[e] = btP[p][e]; }
                        if (e0 == 0) v[0] = l == 0 ? keep : v[0];
#pragma unroll
                        for (int e = e0; e < e0 + EH && e < D::EPL; ++e) {
                            v[e] = e < epl ? x[e] + v[e] : LAST_NEG_INF;
                            m = fmaxf(m, v[e]);
                        }
                        if (D::EPL > 11) __builtin_amdgcn_sched_barrier(0);
                    }
                    m = tri_quad_max(m);
                    const float mm = m == LAST_NEG_INF ? 0.f : m;
                    float z = 0.f;
#pragma unroll
                    for (int e = 0; e < D::EPL; ++e) z += tri_exp(v[e] - mm);
                    z = tri_quad_sum(z);
                    if (l == 0) s.bl[r] = ln_sum(m, z);
                }
                if (D::EPL > 11) __builtin_amdgcn_sched_barrier(0);                // (one row's elements in registers at a time)
            }
            if (!AHEAD) store_row(L - n, a.keep);
            lds_only_barrier();                                                    // B
            if (a.K == 1) lds_only_barrier();
            // (the exchange is under way) the next frame into the tile, the requests for the frame two after it; or the factors of
            // the next frame, the one after it into its tile, the requests for the frame two after that
            if constexpr (AHEAD) {
                const size_t row = a.keep ? (size_t)b * (a.T + 1) + (L - n) : (size_t)b;
                buf_store(rowv, make_buf(a.beta + row * a.C, a.keep ? rowb : 0u), rq, 0);
                nw_store64(rowo, make_buf(a.offb + row, a.keep ? 8u : 0u), oq, 0);
                factors(std::integral_constant<int, Z ^ 1>());
                spread(S);
                issue(S, n + 4);
            } else {
                spread(std::integral_constant<int, Z ^ 1>());
                issue(std::integral_constant<int, Z ^ 1>(), n + 3);
            }
            lds_only_barrier();                                                    // A
        };
        for (int n = 0; n < steps; n += 2) {
            frame(std::integral_constant<int, 0>(), n);
            if (n + 1 < steps) frame(std::integral_constant<int, 1>(), n + 1);
        }
        store_row(L - steps, true);
    } else {
        const int lidx = wave * kWave + lane;
        const bool act = lidx < nbk * V;
        const int pa = act ? lidx / nbk + 1 : 1, pi = act ? lidx - (pa - 1) * nbk : 0;   // published own state
        const int prow = pa * nbk + pi;
        const int gi = act ? lidx / V : 0, gy = act ? lidx - gi * V + 1 : 1;             // gathered state (b0 + gi, gy)
        const bool single = wave == 0 && lane < nbk;
        const bool second = wave == 0 && lane <= nbk;
        const bool starter = o.k == 0 && wave == 0;                                      // gathers the histories of one label
        const int nh = a.K * NCM;
        const unsigned oMine = tri_place((pa - 1) * V + (o.b0 - 1 + pi)), oGot = tri_place((o.b0 - 1) * V + (act ? lidx : 0));
        const unsigned oHead = tri_place(V * V + V + o.k * NCM + wave), oHeads = tri_place(V * V + V + (lane < nh ? lane : 0));
        const unsigned oSingle = tri_place(V * V + (o.b0 - 1 + lane)), oSingles = tri_place(V * V + (lane < V ? lane : 0));
        bool dead = false;
        double A = 0.0;
        __syncthreads();
        for (int n = 0; n < steps; ++n) {
            u64* xs = xbase + (size_t)(gstep & 1) * a.xs;
            const unsigned tag = gstep + 1;
            gstep += 1;
            lds_only_barrier();                                                    // B
            const float val = act ? s.bl[prow] : LAST_NEG_INF;
            const float sv = second && (single || o.k == 0) ? s.bl[single ? lane : o.rows] : LAST_NEG_INF;
            float head = LAST_NEG_INF;
            u64 word = 0, hw = 0;
            float got, gots = LAST_NEG_INF;
            if (a.K == 1) {
                head = tri_wave_max(fmaxf(val, sv));
                if (act) s.xl[(pa - 1) * V + pi] = val;
                if (single) s.xl[V * V + lane] = sv;
                if (lane == 0) s.hd[wave] = head;
                lds_only_barrier();
                got = s.xl[act ? lidx : 0];
                if (starter && lane < V) gots = s.xl[V * V + lane];
                head = s.hd[lane < NCM ? lane : 0];
            } else {
                if (act) xpublish(tri_at(xs, oMine), pack_word(val, tag));
                if (single) xpublish(tri_at(xs, oSingle), pack_word(sv, tag));
                head = tri_wave_max(fmaxf(val, sv));
                if (lane == 0) xpublish(tri_at(xs, oHead), pack_word(head, tag));
                if (!dead) dead = !tri_poll<true, false>(tri_at(xs, oGot), tri_at(xs, oHeads), act, tag,
                                                         a.spin_limit, word, hw);
                got = __uint_as_float((unsigned)word);
                head = __uint_as_float((unsigned)hw);
                if (starter) {
                    if (!dead) dead = !tri_poll<false, false>(tri_at(xs, oSingles), xs, lane < V, tag,
                                                              a.spin_limit, word, hw);
                    gots = __uint_as_float((unsigned)word);
                }
            }
            float mx = tri_wave_max(head);
            if (mx == LAST_NEG_INF) mx = 0.f;
            A += (double)mx;
            if (act) {
                bt[gi * BP + gy] = got - mx;
                if (AHEAD) be[gi * BP + gy] = tri_exp_far(got - mx);
                s.own[prow] = val - mx;
                if (AHEAD) s.ex[prow] = tri_exp_far(val - mx);
            }
            if (starter && lane < V) {
                bt[nbk * BP + 1 + lane] = gots - mx;
                if (AHEAD) be[nbk * BP + 1 + lane] = tri_exp_far(gots - mx);
            }
            if (second && (single || o.k == 0)) {
                s.own[single ? lane : o.rows] = sv - mx;
                if (AHEAD) s.ex[single ? lane : o.rows] = tri_exp_far(sv - mx);
            }
            if (tid == 0) s.off = A;
            if (dead) s.dead = 1;
            lds_only_barrier();                                                    // A
        }
    }
    __syncthreads();
    if (tid == 0 && s.dead) a.fail[b] = 1;
    __syncthreads();
}

// (four waves a SIMD: a cluster of 32 workgroups, a whole XCD, leaves room for that of another launch)
template <typename D, bool TROP>
__global__ __launch_bounds__(D::NW * kWave, 4) void trigram_kernel(TriArgs a)
{
    extern __shared__ __align__(16) float tri_dyn[];
    __shared__ __align__(16) TriLds<D> s;
    // workgroups with equal id % 8 sit on one XCD; a cluster takes K of them per direction.  The directions do not meet
    // in this kernel: those of a cluster with more than 16 workgroups sit on two neighbouring XCDs (across = 1).
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int rx = a.roles >> a.across;
    const int cl = slot / (rx * a.K), rk = slot - cl * rx * a.K;
    const int role = a.across ? xcd & 1 : rk / a.K;
    const int cg = (xcd >> a.across) + (8 >> a.across) * cl;
    TriOwn o;
    o.k = rk % a.K;
    o.V = a.V;
    o.V1 = a.V + 1;
    o.b0 = 1 + o.k * a.nb;
    o.nbk = min(a.nb, a.V - (o.b0 - 1));
    o.W = o.nbk * o.V1;
    o.CQ = (o.W + 3) / 4;
    o.G = a.G;
    o.rows = o.V1 * o.nbk;
    u64* xbase = a.x + (size_t)(cg * a.roles + role) * 2 * a.xs;
    unsigned gstep = 0;
    for (int b = cg; b < a.B; b += (8 >> a.across) * a.ncl) {
        const int L = a.len[b];
        if (L < 0 || L > a.T) continue;
        if (TROP || role == 0) tri_forward<D, TROP>(a, o, b, L, gstep, xbase, s, tri_dyn);
        else tri_backward<D>(a, o, b, L, gstep, xbase, s, tri_dyn);
    }
}

// What the general kernels need to take over an item whose workgroups gave up waiting for each other (their
// partners had no compute unit: other launches of cooperating workgroups share the chip).
struct TriRedo {
    const float* w;
    Ctx c;
    int CPAD, R;         // thread layout of solo_kernels.hpp
    float* dw;           // marginals (may be null)
    float scale;
    int accumulate;
};

// D = log (+)_q alpha_m[q] beta_m[q] of every item from the rows at which the two directions meet (beta = 0 at the
// last frame), one workgroup per item.  alpha, beta: natural logs with offsets.  badtab may be null.
// keep: 0: one row per item; 1: rows of all frames, joined at the last one; 2: rows of all frames, joined where
// keep = 0 joins them, so that the two return the same bits.
// REDO: an item marked in `fail` is computed here once more by this workgroup alone, gradient included
// (dense_marginals_kernel leaves it out; keep = 2: the rows of both directions); dynamic LDS for solo_kernels.hpp.
template <bool REDO>
__global__ __launch_bounds__(256) void tri_join_kernel(
    float* alpha, float* beta, double* offa, double* offb,
    const int* __restrict__ len, const int* __restrict__ fail, const int* __restrict__ badtab, int T, int C, int keep,
    double* D2, float* dist, int* __restrict__ item_status, TriRedo redo)
{
    extern __shared__ float tri_redo_s[];
    __shared__ float red[32];
    __shared__ double redd[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int L = len[b];
    const bool bad = L < 0 || L > T, tab = badtab && badtab[0] != 0;
    if (bad || tab) {
        if (tid == 0) {
            dist[b] = __builtin_nanf("");
            if (D2) D2[b] = __builtin_nan("");
            if (item_status) item_status[b] = tab ? kItemBadTable : kItemBadLength;
        }
        return;
    }
    if (tid == 0 && item_status) item_status[b] = kItemOk;
    if (REDO && fail[b] != 0) {
        solo_forward_item(b, L, tri_redo_s, redo.w, redo.c, T, redo.CPAD, redo.R, keep ? alpha : nullptr,
                          keep ? offa : nullptr, D2, dist);
        __syncthreads();
        if (redo.dw)
            solo_backward_item<16>(b, L, tri_redo_s, redo.w, redo.c, T, alpha, offa, D2, redo.dw, redo.scale, redo.accumulate);
        else if (keep == 2)
            solo_backward_item<16, true>(b, L, tri_redo_s, redo.w, redo.c, T, alpha, offa, D2, nullptr, 0.f, 0, beta, offb);
        return;
    }
    const size_t ra = keep ? (size_t)b * (T + 1) + tri_meet(L, keep == 1) : (size_t)b;
    const bool last = keep == 1;             // (beta is 0 there)
    const float* al = alpha + ra * C;
    const float* be = beta + ra * C;
    float mx = LAST_NEG_INF;
    for (int q = tid; q < C; q += 256) mx = fmaxf(mx, last ? al[q] : al[q] + be[q]);
    mx = block_max(mx, red);
    const float mm = mx == LAST_NEG_INF ? 0.f : mx;
    double z = 0.0;
    for (int q = tid; q < C; q += 256) z += (double)tri_exp((last ? al[q] : al[q] + be[q]) - mm);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
    if ((tid & 63) == 0) redd[tid >> 6] = z;
    __syncthreads();
    if (tid == 0) {
        z = redd[0];
        for (int k = 1; k < 4; ++k) z += redd[k];
        const double d2 = mx == LAST_NEG_INF ? (double)LAST_NEG_INF
                                             : offa[ra] + (last ? 0.0 : offb[ra]) + (double)mm + log(z);
        dist[b] = (float)d2;
        if (D2) D2[b] = d2;
    }
}

// best final state of every item (lowest index among equals) from its final scores; an item marked in `fail` is
// computed here once more by this workgroup alone (dynamic LDS for solo_kernels.hpp)
__global__ __launch_bounds__(256) void tri_final_kernel(
    const float* __restrict__ fin, const int* __restrict__ len, const int* __restrict__ fail, int T, int C,
    int* __restrict__ bp, int* __restrict__ final_state, float* __restrict__ score, int* __restrict__ item_status,
    TriRedo redo)
{
    extern __shared__ float tri_redo_s[];
    __shared__ float redv[4];
    __shared__ int redi[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int L = len[b];
    if (L < 0 || L > T) {
        if (tid == 0) {
            score[b] = __builtin_nanf("");
            if (final_state) final_state[b] = -1;
            if (item_status) item_status[b] = kItemBadLength;
        }
        return;
    }
    if (tid == 0 && item_status) item_status[b] = kItemOk;
    if (fail[b] != 0) {
        solo_viterbi_item(b, L, tri_redo_s, redo.w, redo.c, T, redo.CPAD, redo.R, bp, final_state, score);
        return;
    }
    float best = LAST_NEG_INF;
    int idx = 0x7fffffff;
    for (int q = tid; q < C; q += 256) {
        const float v = fin[(size_t)b * C + q];
        if (v > best || (v == best && q < idx)) { best = v; idx = q; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(idx, o, kWave);
        if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
    }
    if ((tid & 63) == 0) { redv[tid >> 6] = best; redi[tid >> 6] = idx; }
    __syncthreads();
    if (tid == 0) {
        for (int k = 1; k < 4; ++k)
            if (redv[k] > best || (redv[k] == best && redi[k] < idx)) { best = redv[k]; idx = redi[k]; }
        score[b] = best;
        if (final_state) final_state[b] = idx;
    }
}

__global__ void tri_clear_kernel(u64* __restrict__ x, size_t n, int* __restrict__ fail, int B)
{
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = i0; i < n; i += (size_t)gridDim.x * blockDim.x) x[i] = ~0ull;
    for (size_t i = i0; i < (size_t)B; i += (size_t)gridDim.x * blockDim.x) fail[i] = 0;
}

}  // namespace last
