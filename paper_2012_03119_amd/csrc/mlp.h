// Device side of the clause-priority network: a 12 -> 64 -> 64 -> 1 perceptron
// with ReLU hidden layers and a sigmoid output, in fp32.  The paper has no such
// network; it motivates the priority by its Section 3.2 (a clause used recently
// is likely to be used again soon) and Section 3.7 (activity-based deletion on
// the GPU).  Parameters are packed as W1[12][64] (input major), b1[64],
// W2[64][64], b2[64], w3[64], b3: 5057 floats.
//
// Every product runs on the matrix cores in fp32 (v_mfma_f32): the dense fp32 rate
// there is twice the vector units' without packed instructions.
#pragma once

#include "gss_internal.h"

namespace gss {

constexpr int kFeat = 12;
constexpr int kHid = 64;
constexpr int kHist = 8;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kFeat * kHid;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid;
constexpr int kParams = kOffB3 + 1;  // 5057
static_assert(kParams == 5057, "parameter layout");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Inference, 32 samples a wavefront step, with 32x32 outputs and K = 2 per
// instruction on the transposed activations: H1^T = W1^T X^T (K = the 12 features),
// then H2^T = W2^T H1^T (K = the 64 hidden units).  In the 32x32 result a lane holds
// one sample (its column, lane % 32) and 16 rows; those are exactly the values that
// lane must supply as the B operand (one K row for one sample) of the next product,
// so the activations never move between lanes: step s of the second product takes
// its two K rows from register s % 16 of tile s / 16 of the two lane halves, and the
// weights (the A operand) are loaded in that same row order.  The output layer sums
// each lane's 32 rows and its partner lane's (lane ^ 32).  The weights stay in
// registers for all of a wavefront's steps, the biases and output weights in LDS.

// row of the 32x32 result held in register v by a lane of half `half`
__device__ constexpr uint32_t mfma_row(uint32_t v, uint32_t half) { return 8 * (v / 4) + 4 * half + (v % 4); }

struct MlpBiases {  // in LDS
    float b1[kHid], b2[kHid], w3[kHid];
    __device__ void load(const float *__restrict__ p) {  // by a workgroup; a barrier follows
        for (uint32_t t = threadIdx.x; t < kHid; t += blockDim.x) {
            b1[t] = p[kOffB1 + t];
            b2[t] = p[kOffB2 + t];
            w3[t] = p[kOffW3 + t];
        }
    }
};

struct MlpWeights {  // one lane's operands
    float w1a[2][kFeat / 2], w2a[2][kHid / 2], b3;
    __device__ void load(const float *__restrict__ p, uint32_t half, uint32_t col) {
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) {
#pragma unroll
            for (uint32_t st = 0; st < kFeat / 2; ++st) w1a[u][st] = p[kOffW1 + (2 * st + half) * kHid + 32 * u + col];
#pragma unroll
            for (uint32_t st = 0; st < kHid / 2; ++st) {
                const uint32_t hid = 32 * (st / 16) + mfma_row(st % 16, half);
                w2a[u][st] = p[kOffW2 + hid * kHid + 32 * u + col];
            }
        }
        b3 = p[kOffB3];
    }
};

// The output logit of the lane's sample (both halves of the wavefront get it).
// xh[st]: feature 2 st + half of sample `col`.
__device__ inline float mlp_tile_logit(const MlpWeights &w, const MlpBiases &s, const float (&xh)[kFeat / 2],
                                       uint32_t half) {
    // an index the compiler cannot see through: the LDS reads stay in the
    // caller's loop instead of being hoisted into 96 more registers per lane
    uint32_t lds_row = 4 * half;
    asm volatile("" : "+v"(lds_row));
    f32x16 acc1[2], acc2[2];
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u)
#pragma unroll
        for (uint32_t v = 0; v < 16; ++v) {
            const uint32_t row = 32 * u + 8 * (v / 4) + (v % 4) + lds_row;  // mfma_row(v, half)
            acc1[u][v] = s.b1[row];
            acc2[u][v] = s.b2[row];
        }
#pragma unroll
    for (uint32_t st = 0; st < kFeat / 2; ++st)
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u)
            acc1[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.w1a[u][st], xh[st], acc1[u], 0, 0, 0);
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u)
#pragma unroll
        for (uint32_t v = 0; v < 16; ++v) acc1[u][v] = fmaxf(acc1[u][v], 0.f);
#pragma unroll
    for (uint32_t st = 0; st < kHid / 2; ++st) {
        const float bh = acc1[st / 16][st % 16];
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u)
            acc2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.w2a[u][st], bh, acc2[u], 0, 0, 0);
    }
    float part = 0.f;
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u)
#pragma unroll
        for (uint32_t v = 0; v < 16; ++v)
            part = fmaf(fmaxf(acc2[u][v], 0.f), s.w3[32 * u + 8 * (v / 4) + (v % 4) + lds_row], part);
    return part + __shfl_xor(part, 32) + w.b3;
}

__device__ inline float sigmoidf_(float z) { return 1.f / (1.f + expf(-z)); }

// softplus(z) - y z: the binary cross-entropy of logit z against label y.
__device__ inline float bce_logit(float z, float y) { return fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - y * z; }

// The 12 features of a clause from its raw statistics: length, LBD, age in runs,
// source thread, hit counts of its last 8 tested runs (most recent first).
__device__ inline void clause_features(float (&x)[kFeat], uint32_t len, float lbd, uint32_t age, uint32_t src,
                                       float src_scale, const uint32_t (&hist)[kHist]) {
    x[0] = log1pf((float)len);
    x[1] = log1pf(lbd);
    x[2] = log1pf((float)age);
    x[3] = (float)src * src_scale;
#pragma unroll
    for (int k = 0; k < kHist; ++k) x[4 + k] = log1pf((float)hist[k]);
}

// Host-side workspace of the network's kernels (one per context, grown on demand).
struct MlpWork {
    float *params = nullptr;  // [kParams]
    float *m = nullptr, *v = nullptr, *grad = nullptr;  // Adam moments, reduced gradient
    float *partials = nullptr;  // [blocks][kParams + 1] (the last entry of a row: loss)
    uint32_t partial_rows = 0;
    float *loss = nullptr;      // [1]
    char *stage = nullptr;      // device copies of host inputs
    size_t stage_bytes = 0;
    float *h_loss = nullptr;    // pinned
    uint64_t step = 0;          // Adam steps taken with the current moments
};

constexpr uint32_t kGradSamples = 16;  // samples per group of the gradient kernel
constexpr uint32_t kGradBlocks = 256;  // its workgroups at most, each with a partial gradient

// Queues the gradient of the mean loss over n samples (rows order[first..first+n)
// of x/y, or rows first..first+n when order is null) into w.grad, its loss into
// w.loss; inv_n scales both.
void mlp_queue_grad(Ctx &c, MlpWork &w, const float *x, const float *y, const uint32_t *order, uint64_t first,
                    uint32_t n);
// Queues the same gradient and one Adam step on w.params from it; the loss goes to
// *loss (device).
void mlp_queue_step(Ctx &c, MlpWork &w, const float *x, const float *y, const uint32_t *order, uint64_t first,
                    uint32_t n, float lr, float beta1, float beta2, float eps, float *loss);
// Workgroups of 4 wavefronts for inference on n samples, 32 per wavefront step; at
// most 2 workgroups per compute unit, as many as are resident with the weights in
// registers (4 M samples in 362 us a call; with 1 411, with 3 373, with 4 361).
unsigned mlp_grid(const Ctx &c, uint64_t n);
MlpWork &mlp_work(Ctx &c);
void mlp_release(Ctx &c);
char *mlp_stage(Ctx &c, MlpWork &w, size_t bytes);

}  // namespace gss
