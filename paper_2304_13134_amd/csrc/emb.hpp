// Lattices of two-label contexts with shared-embedding weights
//     w[t][q][:] = bf16(tanh(f[t] + e[q])) @ W        (arXiv 2304.13134, Section 4.1)
// whose weights are laid out in memory frame by frame for the recursions of trigram_kernels.hpp: plans and
// launches (emb_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace last {

constexpr int kEmTile = 32;          // states of a tile
constexpr int kEmMaxLabelTiles = 5;  // V + 1 <= 80 in tiles of 16
constexpr int kEmScan = 1024;        // workgroups that go over f and e

struct EmbArgs {
    const void *f, *e, *W;           // bfloat16 [B][T][H], [C][H], [H][V+1]
    const int* len;
    float *Ef, *Ee;                  // [B T][H], [tiles 32][H]: e^2f, e^2e
    void* Wn;                        // W as operand fragments of the weights
    void* Wt;                        // W transposed as operand fragments of the gradient
    int2* frames;                    // (row b T + t, item b) of the frames that exist, item by item
    int* count;                      // how many
    int* big;                        // per such workgroup: large values in f (1), in e (2)
    float* w;                        // [B][T][C][V+1]
    unsigned long long* x;           // exchange area and flags of the recursions, cleared on the way
    size_t xwords;
    int* fail;
    int B, T, C, V, H;
    int tiles;                       // ceil(C / 32)
    int nch;                         // stretches of frames of the weights kernel
};

struct EmbNorm {                     // of a frame t: ln of the scale of alpha_t + beta_{t+1}, 1 / partition sum
    double k;
    float iz, unused;
};

// The gradient pass.  alpha, beta [B][T+1][C] natural logarithms relative to offa, offb [B][T+1].
struct EmbGradArgs {
    const float *alpha, *beta;
    const double *offa, *offb;
    EmbNorm* norm;                   // [B T]
    // marginals of the intersected lattice (null: none), [B T][U1] (empty label, label), and its cells by tile
    const float2* pn;
    const int *cells, *starts;       // [B][U1] u << 12 | state in the tile << 7 | label; [B][tiles + 1]
    int U1;
    float *pdf, *pde, *pdw;          // partial sums [tiles][B T][H], [ngr][tiles 32][H], [ngr tiles][H][V+1]
    int ngr;                         // stretches of frames
    float *df, *de, *dW;
    float scale;
    int acc_df, acc_rest;            // add to what is there
};

// numerator of a loss: what numerator_kernels.hpp left, for the items of the workspace
struct EmbNumArgs {
    float2* wi;                      // [B][T][U1] weights, overwritten with the marginals
    const double *a, *bk, *N;        // [B][T+1][U1] twice, [B]
    const int *status, *ctxs, *refs, *ulen;
    int *cells, *starts;
    int U1;
};

struct EmbPlan {
    bool ok;
    int tiles, nch, ngr;
    size_t row;                      // bytes of the weights of a frame
    size_t lds;
};

// B, T: of the items that are in the workspace at a time
EmbPlan emb_plan(int B, int T, int C, int V, int H);
// workgroups of one launch in stretches of frames: so many stretches that the last round over the chip is well filled
int emb_stretches(int tiles, size_t frames, int shortest, int startup);
hipError_t emb_launch_weights(const EmbArgs& a, const EmbPlan& p, hipStream_t st);
hipError_t emb_launch_numerator(const EmbArgs& a, const EmbNumArgs& n, hipStream_t st);
hipError_t emb_launch_gradient(const EmbArgs& a, const EmbGradArgs& g, hipStream_t st);

}  // namespace last
