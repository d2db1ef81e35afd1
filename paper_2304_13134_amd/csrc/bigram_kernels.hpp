// Full 1-gram contexts of 66 to 96 states with dense weights: one
// workgroup per item and direction, no exchange between compute units.
// (Up to 65 states the chain of frames runs in one wavefront, bigram_wave_kernels.hpp, with the arithmetic and the
// joining kernel that are described here; paths and distances of many items stay here, see bw_ok in last_api.hip.)
//
// A frame is a C x C matrix; at these sizes one compute unit can stream it and
// the recursions (Eq. 2 of arXiv 2304.13134, both directions, and the tropical
// one of Section 4.2.3) are bound by the chain of a frame: matrix-vector
// product -> LDS -> barrier -> new vector -> normalisation.  A cluster of
// workgroups pays an exchange through L2 on top of that, 2.5 to 3 us a frame.
//
// Half of the waves ("producers") fetch the weights with 16-byte loads, LPR
// lanes a row, and turn them into E = 2^(w log2 e - s_q) <= 1 with an integer
// shift s_q >= max_y w[q][y] log2 e per row, two frames ahead of the recursion,
// through LDS.  The other half ("consumers") run the recursion: wave <-> rows
// [wave rc, (wave + 1) rc), lane <-> column (64 CB of them); every one of them
// keeps the whole state vector in its lanes, so that a row's state is a readlane
// away, and requests the E of its next frame from LDS before the barrier:
//   forward : partial column sums of the wave's rows -> LDS -> added up in wave order;
//   backward: products of the rows with the vector, reduced over the lanes eight
//             rows at a time (three steps that merge two rows each, three adds), row sums -> LDS;
//   tropical: as forward with (score, source row) and first-maximum rules.
// Arithmetic is scaled linear float32: the state vector is brought to
// 2^(s_q - S + 100) state_q with S the largest exponent present, the exponents S - 100 add up
// in a float64 offset per frame, and a sum of 97 products stays below 2^108.  What is lost is what
// lies 2^126 below the largest weight of its row or 2^226 below the largest state of its
// frame: nothing to a sum, unless paths make up for it elsewhere.  With marginals an item that may have
// lost a part is flagged (marginals_kernels.hpp).  Without them the consumers note
//  - whether a frame with a state so small that lost weights could have been a part of it (below kBiThin; they are
//    below 2^-18 together) was followed by one that does not bury them again: in which a state is not above
//    kBiThick, or a row's weights are more than 2^20 above those of the states that matter;
//  - whether states that may be lost as a factor (kBiSmall) came before a frame that does not bury them.
// bigram_join_kernel looks through the weights of the former items for some that are far below their row's largest,
// computes those and the latter in the log domain, and so the distance is exact but for two things
// that count as absent: weights more than 1040 below the largest of their row, and paths that stay in the
// start state (which nothing leads back to, so that it always falls behind) until they are 2^226
// behind and make up for that later.
// (What was tried instead: E with a span of 2^176, 7 vector instructions a weight instead of 2, the loss at 8
// items, 200 frames, 32 labels 193 us instead of 177; the weights tested by the producers, the distance 95
// instead of 84 us.  The producers are the longer half of a frame.)
// Marginals are formed afterwards from the stored vectors (marginals_kernels.hpp).
//
// Measured: figures beside bi_ok in last_api.hip.  Loops over a wave's rows run
// over all RC of them: with a test per row the compiler kept every row's state alive
// along every path and spilled by the thousand.
#pragma once
#include "cluster_kernels.hpp"
#include "common.hpp"
#include "numerator_kernels.hpp"
#include "solo_kernels.hpp"
#include "trigram_kernels.hpp"

namespace last {

struct BiArgs {
    const float* w;
    const int* len;
    float* alpha;        // rows of C floats, relative to 2^offset; tropical: unused
    float* beta;
    double* offa;
    double* offb;
    double* D2;          // KEEP: base-2 logarithm of the partition sum
    float* dist;
    int* item_status;
    int* bp;             // tropical: [B][T][C] flat arc indices (may be null)
    int* final_state;
    int T, C, P;         // P: pitch of E in LDS, C rounded up to 4
    int rc, rp;          // rows per consumer, rows per producer
    int* wide;           // not KEEP: [B][2], 1: weights may have been lost, 2: states may have been
};

constexpr int kBiMaxC = 96;
constexpr int kBiCentre = 100;           // exponent of the largest state
constexpr float kBiThin = 1024.f;                    // 2^10
constexpr float kBiThick = 1.1529215e18f;            // 2^60: what a thin state has lost is 2^-51 of the states after it
constexpr int kBiOver = 20;
constexpr unsigned kBiAbsent = 1500, kBiSmall = 1340;    // states 2^160 to 2^1500 below the largest (kBiAbsent less is the unit)
constexpr float kBiFar = 60.f;                       // weights that may be lost against such a state: 2^60 to 2^1500 below
                                                     // their row's largest; beyond 2^1500 they are meant to

// Sum or maximum over the 64 lanes of R = 8 or 4 rows at a time; lane l ends with row bi_row<R>(l).
template <int R>
__device__ __forceinline__ int bi_row(int l)
{
    return R == 8 ? ((l >> 5) & 1) * 4 + ((l >> 4) & 1) * 2 + ((l >> 3) & 1) : ((l >> 5) & 1) * 2 + ((l >> 4) & 1);
}
template <bool MAX>
__device__ __forceinline__ float bi_op(float x, float y) { return MAX ? fmaxf(x, y) : x + y; }
template <bool MAX>
__device__ __forceinline__ float bi_merge32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return bi_op<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <bool MAX>
__device__ __forceinline__ float bi_merge16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return bi_op<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int R, bool MAX>
__device__ __forceinline__ float bi_rows(const float* v, int lane)
{
    float y;
    if (R == 8) {
        const float u0 = bi_merge32<MAX>(v[0], v[4]), u1 = bi_merge32<MAX>(v[1], v[5]);
        const float u2 = bi_merge32<MAX>(v[2], v[6]), u3 = bi_merge32<MAX>(v[3], v[7]);
        const float x0 = bi_merge16<MAX>(u0, u2), x1 = bi_merge16<MAX>(u1, u3);
        const bool hi = lane & 8;
        const float keep = hi ? x1 : x0, send = hi ? x0 : x1;
        y = bi_op<MAX>(keep, dpp_f<0x128>(send, send));            // row_ror:8
    } else {
        const float u0 = bi_merge32<MAX>(v[0], v[2]), u1 = bi_merge32<MAX>(v[1], v[3]);
        const float x0 = bi_merge16<MAX>(u0, u1);
        y = bi_op<MAX>(x0, dpp_f<0x128>(x0, x0));
    }
    y = bi_op<MAX>(y, dpp_f<0x141>(y, y));                         // row_half_mirror
    y = bi_op<MAX>(y, dpp_f<0xB1>(y, y));                          // quad_perm 1,0,3,2
    return bi_op<MAX>(y, dpp_f<0x4E>(y, y));                       // quad_perm 2,3,0,1
}

__device__ __forceinline__ float bi_readlane(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// LPR: lanes per row of a producer; CB: columns per lane / 64 of a consumer; NC consumers, NP producers; RC: most
// rows of a consumer (a multiple of 4); PP: 16-byte pieces of a frame per producer lane; DS: frames requested ahead
template <int LPR_, int CB_, int NC_, int NP_, int RC_, int PP_, int DS_>
struct BiDims {
    static constexpr int LPR = LPR_, CB = CB_, NC = NC_, NP = NP_, RC = RC_, PP = PP_, DS = DS_;
    static constexpr int N = 64 * CB, Rows = NC * RC > NP * PP * (64 / LPR) ? NC * RC : NP * PP * (64 / LPR);
};

template <typename D, bool TROP>
struct BiLds {
    float part[2][D::NC][D::N];                      // forward: partial sums; tropical: scores
    unsigned char src[TROP ? 2 : 1][TROP ? D::NC : 1][D::N];   // tropical: row of the wave
    float rs[2][D::Rows];                            // backward: row sums
    int sv[4][D::Rows];                              // row shifts, by step mod 4
    float e0[4][D::Rows];                            // E (tropical: weight) of the empty label, by step mod 4
};

// grid (B, roles): blockIdx.y = 0 forward, 1 backward.  Dynamic LDS: E [2][C][P].
// KEEP: every row at [b][T+1][C], distance written; else the meeting row at [b][C].
template <typename D, bool TROP, bool KEEP>
__global__ __launch_bounds__((D::NC + D::NP) * 64) void bigram_kernel(BiArgs a)
{
    constexpr int CB = D::CB, NC = D::NC, RC = D::RC, PP = D::PP, LPR = D::LPR, RPP = 64 / LPR, DS = D::DS;
    extern __shared__ __align__(16) float bi_E[];
    __shared__ __align__(16) BiLds<D, TROP> s;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool back = !TROP && blockIdx.y == 1;
    const int C = a.C, P = a.P, L = a.len[b];
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
    const int esz = C * P;
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;

    if (wave >= NC) {
        // ------------------------------------------------------------ producer
        if (steps == 0) return;
        const size_t fr = (size_t)C * C;
        const float* wi = a.w + (size_t)b * a.T * fr;
        const int q0 = (wave - NC) * a.rp;                      // own rows q0 .. q0 + rp - 1
        const int lq = lane / LPR, lc = lane - lq * LPR;
        const int piece = min(lc, P / 4 - 1);                   // lanes beyond the row repeat its last piece
        const unsigned frb = 4u * (unsigned)fr;
        // a row's last piece ends with it: it holds columns C - 4 .. C - 1 at places P - 4 .. P - 1
        const int c0 = min(4 * piece, C - 4);
        float4 raw[DS][PP];
        auto row_of = [&](int p) __attribute__((always_inline)) { return q0 + p * RPP + lq; };
        auto issue = [&](auto S, int n) __attribute__((always_inline)) {
            const int t = back ? max(L - 1 - n, 0) : min(n, L - 1);
            const buf_t rs = make_buf(wi + (size_t)t * fr, frb);
#pragma unroll
            for (int p = 0; p < PP; ++p)
                raw[decltype(S)::value][p] = tri_load4(rs, 4u * (unsigned)(min(row_of(p), C - 1) * C + c0), 0);
        };
        // step n out of its requested pieces, and the request for step n + DS
        auto prep = [&](auto S, int n) __attribute__((always_inline)) {
            constexpr int Z = decltype(S)::value;
            float* eb = bi_E + (n & 1) * esz;
#pragma unroll
            for (int p = 0; p < PP; ++p) {
                float4 w = raw[Z][p];
                const int q = row_of(p);
                const bool mine = p * RPP + lq < a.rp && q < C;
                if (!TROP) {
                    float m = fmaxf(fmaxf(w.x, w.y), fmaxf(w.z, w.w));
                    // over the lanes of the row
                    if (LPR >= 32) {
                        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
                        m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
                    }
                    if (LPR >= 16) m = fmaxf(m, dpp_f<0x128>(m, m));
                    m = fmaxf(m, dpp_f<0x141>(m, m));
                    m = fmaxf(m, dpp_f<0xB1>(m, m));
                    m = fmaxf(m, dpp_f<0x4E>(m, m));
                    const int sh = shift_for(m);
                    const float ns = -(float)sh;
                    w.x = fast_exp2(fmaf(w.x, kLog2e, ns));
                    w.y = fast_exp2(fmaf(w.y, kLog2e, ns));
                    w.z = fast_exp2(fmaf(w.z, kLog2e, ns));
                    w.w = fast_exp2(fmaf(w.w, kLog2e, ns));
                    if (mine && lc == 0) s.sv[n & 3][q] = sh;
                }
                if (mine && lc == 0) s.e0[n & 3][q] = w.x;
                if (mine && lc < P / 4) *(float4*)(eb + q * P + 4 * lc) = w;
            }
            issue(S, n + DS);
        };
        issue(I0(), 0);
        if (DS == 2) issue(std::integral_constant<int, DS - 1>(), 1);
        prep(I0(), 0);
        prep(std::integral_constant<int, DS - 1>(), 1);
        lds_only_barrier();
        lds_only_barrier();                                     // (the consumers have E of step 0: step 2 goes to its place)
        for (int t = 0; t < steps; t += 2) {
            prep(I0(), t + 2);
            lds_only_barrier();
            if (t + 1 >= steps) break;
            prep(std::integral_constant<int, DS - 1>(), t + 3);
            lds_only_barrier();
        }
        return;
    }

    // ---------------------------------------------------------------- consumer
    const int q0 = wave * a.rc;                                 // own rows q0 .. q0 + nr - 1
    const int nr = max(min(a.rc, C - q0), 0);
    // columns beyond the matrix repeat the last one; they meet a zero (tropical: -inf) state in every sum
    int col[CB], place[CB];
    bool ok[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        ok[c] = 64 * c + lane < C;
        col[c] = min(64 * c + lane, C - 1);
        place[c] = col[c] + (col[c] >= P - 4 ? P - C : 0);
    }
    float E[RC][CB];
    auto fetch = [&](int n) __attribute__((always_inline)) {    // (rows beyond the own ones repeat the last)
        const float* eb = bi_E + (n & 1) * esz;
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const float* row = eb + min(q0 + min(r, max(nr, 1) - 1), C - 1) * P;
#pragma unroll
            for (int c = 0; c < CB; ++c) E[r][c] = row[place[c]];
        }
    };
    float v[CB];                                     // the state vector, lane <-> state
    double A = 0.0;
    // not KEEP: exponents of the positive states below the largest one's, from kBiAbsent down; a lane without a state, and
    // the start state in the forward direction, do not count
    unsigned small[CB];
    bool was_thin = false, unburied = false, unburied_small = false;
    float not_thin[CB];
    unsigned not_small[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const bool out = !ok[c] || (!back && c == 0 && lane == 0);
        not_thin[c] = out ? __builtin_inff() : 0.f;
        not_small[c] = out ? ~0u : 0u;
        small[c] = ~0u;
    }
    auto look = [&]() __attribute__((always_inline)) {                  // at the new states
        float least = v[0] + not_thin[0];
#pragma unroll
        for (int c = 1; c < CB; ++c) least = fminf(least, v[c] + not_thin[c]);
        if (!__any(least < kBiThick)) {
            was_thin = false;
            return;
        }
        unsigned s0 = small[0];
#pragma unroll
        for (int c = 1; c < CB; ++c) s0 = min(s0, small[c]);
        unburied = unburied || was_thin;
        unburied_small = unburied_small || __any(s0 < kBiSmall);
        was_thin = __any(least < kBiThin);
    };
    auto note = [&]() __attribute__((always_inline)) {
        if (KEEP || wave != 0) return;
        const int f = (unburied ? 1 : 0) | (unburied_small ? 2 : 0);
        if (lane == 0) a.wide[(size_t)b * 2 + (back ? 1 : 0)] = f;
    };
    auto put_row = [&](float* base, double* off, int t) __attribute__((always_inline)) {
        if (wave != 0) return;
        const size_t row = KEEP ? (size_t)b * (a.T + 1) + t : (size_t)b;
#pragma unroll
        for (int c = 0; c < CB; ++c)
            if (ok[c]) base[row * C + 64 * c + lane] = v[c];
        if (lane == 0) off[row] = A;
    };
    // state of own row r as a uniform value; 0 (tropical: -inf) beyond the last
    auto own_state = [&](const float (&x)[CB], int r) __attribute__((always_inline)) {
        const int q = q0 + r;
        float y = bi_readlane(x[0], q & 63);
#pragma unroll
        for (int c = 1; c < CB; ++c) {
            const float z = bi_readlane(x[c], q & 63);
            y = q >= 64 * c ? z : y;
        }
        return r < nr ? y : (TROP ? LAST_NEG_INF : 0.f);
    };
    // 2^(s_q - S) v_q with S the largest exponent present; returns S
    auto normalise = [&](const int (&sh)[CB], float (&x)[CB]) __attribute__((always_inline)) {
        int top = -0x40000000, ex[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            ex[c] = v[c] > 0.f ? float_exponent(v[c]) + sh[c] : -0x40000000;
            top = max(top, ex[c]);
        }
        top = wave_max_dpp(top);
        if (top == -0x40000000) top = 0;             // no state reachable
#pragma unroll
        for (int c = 0; c < CB; ++c) x[c] = __builtin_ldexpf(v[c], sh[c] - top + kBiCentre);
        if (!KEEP) {
#pragma unroll
            for (int c = 0; c < CB; ++c) small[c] = (unsigned)(ex[c] - (top - (int)kBiAbsent)) | not_small[c];
            if (was_thin) {
                int most = sh[0];
#pragma unroll
                for (int c = 1; c < CB; ++c) most = max(most, sh[c]);
                unburied = unburied || __any(most - top + kBiCentre > kBiOver);
            }
        }
        return top - kBiCentre;
    };

    if (steps > 0) {
        lds_only_barrier();
        fetch(0);
        lds_only_barrier();
    }

    if (TROP) {
#pragma unroll
        for (int c = 0; c < CB; ++c) v[c] = c == 0 && lane == 0 ? 0.f : LAST_NEG_INF;
        auto frame = [&](auto PAR, int t) __attribute__((always_inline)) {
            constexpr int Z = decltype(PAR)::value;
            float best[CB], w0[CB];
            int src[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) { best[c] = LAST_NEG_INF; src[c] = 255; }
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                const float x = own_state(v, r);
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    const float y = __fadd_rn(x, E[r][c]);
                    const bool up = y > best[c];                   // ascending rows: the first maximum stays
                    best[c] = up ? y : best[c];
                    src[c] = up ? r : src[c];
                }
            }
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                s.part[Z][wave][64 * c + lane] = best[c];
                s.src[Z][wave][64 * c + lane] = (unsigned char)src[c];
                w0[c] = s.e0[t & 3][col[c]];
            }
            fetch(t + 1);
            lds_only_barrier();
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const int y = 64 * c + lane;
                float x = LAST_NEG_INF, z[NC];
                int f = 0, g[NC];
#pragma unroll
                for (int k = 0; k < NC; ++k) { z[k] = s.part[Z][k][y]; g[k] = s.src[Z][k][y]; }
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    f = z[k] > x ? k * a.rc + g[k] : f;
                    x = z[k] > x ? z[k] : x;
                }
                // the label candidate against the empty label, which keeps the state: higher score, then lower arc
                const float xb = __fadd_rn(v[c], w0[c]);
                int fl = f * C + y, fb = y * C;
                if (y == 0) x = LAST_NEG_INF;                      // (column 0 is the empty label)
                if (x == LAST_NEG_INF) fl = 0x7fffffff;
                if (xb == LAST_NEG_INF) fb = 0x7fffffff;
                const bool first = x > xb || (x == xb && fl < fb);
                v[c] = ok[c] ? (first ? x : xb) : LAST_NEG_INF;
                const int flat = first ? fl : fb;
                if (wave == 0 && a.bp && ok[c]) a.bp[((size_t)b * a.T + t) * C + y] = flat == 0x7fffffff ? -1 : flat;
            }
        };
        for (int t = 0; t < steps; t += 2) {
            frame(I0(), t);
            if (t + 1 < steps) frame(I1(), t + 1);
        }
        if (wave == 0) {
            // best final state, lowest index among equals
            float best = LAST_NEG_INF;
            int idx = 0x7fffffff;
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (ok[c] && (v[c] > best || (v[c] == best && 64 * c + lane < idx))) { best = v[c]; idx = 64 * c + lane; }
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
        }
        return;
    }

    if (!back) {
#pragma unroll
        for (int c = 0; c < CB; ++c) v[c] = c == 0 && lane == 0 ? 1.f : 0.f;
        auto frame = [&](auto PAR, int t) __attribute__((always_inline)) {
            constexpr int Z = decltype(PAR)::value;
            int sh[CB];
            float x[CB], eb[CB], acc[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                sh[c] = s.sv[t & 3][col[c]];
                eb[c] = s.e0[t & 3][col[c]];
                acc[c] = 0.f;
            }
            if (KEEP) put_row(a.alpha, a.offa, t);
            const int top = normalise(sh, x);
            A += (double)top;
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                const float q = own_state(x, r);
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[c] = fmaf(q, E[r][c], acc[c]);
            }
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                s.part[Z][wave][64 * c + lane] = acc[c];
                eb[c] *= x[c];                                     // the empty label keeps the state
            }
            fetch(t + 1);
            lds_only_barrier();
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                float y = 0.f, z[NC];
#pragma unroll
                for (int k = 0; k < NC; ++k) z[k] = s.part[Z][k][64 * c + lane];
#pragma unroll
                for (int k = 0; k < NC; ++k) y += z[k];
                if (c == 0 && lane == 0) y = 0.f;                  // (column 0 is the empty label)
                v[c] = ok[c] ? y + eb[c] : 0.f;
            }
            if (!KEEP) look();
        };
        for (int t = 0; t < steps; t += 2) {
            frame(I0(), t);
            if (t + 1 < steps) frame(I1(), t + 1);
        }
        put_row(a.alpha, a.offa, steps);
        note();
        if (KEEP && wave == 0) {
            // all states of the last frame are final with weight 0
            double z = 0.0;
#pragma unroll
            for (int c = 0; c < CB; ++c) z += (double)v[c];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
            if (lane == 0) {
                const double d2 = A + log2(z);
                a.D2[b] = d2;
                a.dist[b] = (float)(d2 * 0.6931471805599453);
                if (a.item_status) a.item_status[b] = kItemOk;
            }
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) v[c] = ok[c] ? __builtin_ldexpf(1.f, kBiCentre) : 0.f;
    A = -(double)kBiCentre;
    if (KEEP || steps == 0) put_row(a.beta, a.offb, L);
    auto frame = [&](auto PAR, int n) __attribute__((always_inline)) {
        constexpr int Z = decltype(PAR)::value;
        float p[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            // column 0 is the empty label: it leads back to the row's own state
            const float own = own_state(v, r);
            p[r] = E[r][0] * (lane == 0 ? own : v[0]);
#pragma unroll
            for (int c = 1; c < CB; ++c) p[r] = fmaf(E[r][c], v[c], p[r]);
        }
        fetch(n + 1);
#pragma unroll
        for (int r0 = 0; r0 < RC; r0 += 8) {
            const bool eight = RC - r0 >= 8;
            const float y = eight ? bi_rows<8, false>(p + r0, lane) : bi_rows<4, false>(p + r0, lane);
            const int row = r0 + (eight ? bi_row<8>(lane) : bi_row<4>(lane));
            if (row < nr && (lane & 7) == 0) s.rs[Z][q0 + row] = y;
        }
        lds_only_barrier();
        int sh[CB];
        float x[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            sh[c] = s.sv[n & 3][col[c]];
            v[c] = s.rs[Z][col[c]];
            v[c] = ok[c] ? v[c] : 0.f;
        }
        if (!KEEP) look();
        const int top = normalise(sh, x);
        A += (double)top;
#pragma unroll
        for (int c = 0; c < CB; ++c) v[c] = x[c];
        if (KEEP || n + 1 == steps) put_row(a.beta, a.offb, L - 1 - n);
    };
    for (int n = 0; n < steps; n += 2) {
        frame(I0(), n);
        if (n + 1 < steps) frame(I1(), n + 1);
    }
    note();
}

// D = log2 sum_q alpha_m[q] beta_m[q] of every item at the frame where the two directions meet (the call without
// marginals).  An item some part of which may have been lost (`wide`, after a look through its weights; or the sum more than
// 2^60 below the product of the two maxima, so that states lost from one vector may matter in the other)
// is computed with the general recursion (dynamic LDS of solo_layout).
__global__ __launch_bounds__(1024) void bigram_join_kernel(
    const float* __restrict__ w, Ctx c, int CPAD, int R, const float* __restrict__ alpha, const float* __restrict__ beta,
    const double* __restrict__ offa, const double* __restrict__ offb, const int* __restrict__ wide,
    const int* __restrict__ len, int T, float* __restrict__ dist, int* __restrict__ item_status)
{
    extern __shared__ float bi_join_s[];
    __shared__ int apart, thin, found;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
    const int L = len[b];
    if (L < 0 || L > T) {
        if (tid == 0) {
            dist[b] = __builtin_nanf("");
            if (item_status) item_status[b] = kItemBadLength;
        }
        return;
    }
    if (tid < kWave) {
        double z = 0.0;
        float am = 0.f, bm = 0.f;
        for (int q = tid; q < c.C; q += kWave) {
            const float x = alpha[(size_t)b * c.C + q], y = beta[(size_t)b * c.C + q];
            z += (double)x * (double)y;
            am = fmaxf(am, x);
            bm = fmaxf(bm, y);
        }
        const int f = wide[(size_t)b * 2] | wide[(size_t)b * 2 + 1];
        am = wave_max_dpp(am);
        bm = wave_max_dpp(bm);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
        if (tid == 0) {
            const double lz = log2(z);
            dist[b] = (float)((offa[b] + offb[b] + lz) * 0.6931471805599453);
            if (item_status) item_status[b] = kItemOk;
            apart = (f & 2) || (am > 0.f && bm > 0.f
                                && (double)(__builtin_amdgcn_logf(am) + __builtin_amdgcn_logf(bm)) - lz > 60.0);
            thin = f & 1;
            found = 0;
        }
    }
    __syncthreads();
    if (!apart && thin) {
        // (a row per wave, eight rows in flight; rows are at most 128 long)
        const float* wi = w + (size_t)b * T * c.C * c.V1;
        const int rows = L * c.C, last = c.V1 - 1, c0 = min(lane, last), c1 = min(lane + kWave, last);
        constexpr int NW = 1024 / kWave, U = 8;
        bool far = false;
        for (int r0 = tid / kWave; r0 < rows; r0 += NW * U) {
            float x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float* row = wi + (size_t)min(r0 + NW * u, rows - 1) * c.V1;
                x[u] = row[c0];
                y[u] = row[c1];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float ns = -(float)shift_for(wave_max_dpp(fmaxf(x[u], y[u])));
                const float p = fmaf(x[u], kLog2e, ns), q = fmaf(y[u], kLog2e, ns);
                far = far || (p < -kBiFar && p > -(float)kBiAbsent) || (q < -kBiFar && q > -(float)kBiAbsent);
            }
        }
        if (far) found = 1;
        __syncthreads();
    }
    if (apart || found) solo_forward_item(b, L, bi_join_s, w, c, T, CPAD, R, nullptr, nullptr, nullptr, dist);
}

}  // namespace last
