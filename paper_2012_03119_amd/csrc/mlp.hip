// Kernels and entry points of the clause-priority network (mlp.h): batched
// inference, the gradient of the mean binary cross-entropy, and Adam.
#include "mlp.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>

namespace gss {

// 32 samples a wavefront step (mlp_tile_logit); the next step's features are loaded
// while the current one multiplies.  Bound by the fp32 matrix rate: 76 instructions
// of 64 cycles for 32 samples, 31 us for 500 K samples on 1024 SIMDs at 2.4 GHz.
// 500 K samples: 56 us (a sample a lane with fp32 vector multiply-adds and scalar
// weights: 100 us); the call 121 -> 74 us, with 1000 samples 81 -> 30 us.
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ p, const float *__restrict__ x,
                                                     uint32_t n, float *__restrict__ out) {
    __shared__ MlpBiases bias;
    bias.load(p);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    MlpWeights w;
    w.load(p, half, col);
    const uint64_t step = (uint64_t)gridDim.x * (blockDim.x / 64) * 32;
    uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64) * 32;
    // past the end a lane reads the last sample's features and stores nothing
    auto features = [&](uint64_t b, float (&v)[kFeat / 2]) {
        const float *src = x + min(b + col, (uint64_t)n - 1) * kFeat + half;
#pragma unroll
        for (uint32_t st = 0; st < kFeat / 2; ++st) v[st] = src[2 * st];
    };
    float cur[kFeat / 2];
    features(base, cur);
    for (; base < n; base += step) {
        float nxt[kFeat / 2];
        features(base + step, nxt);
        const float z = mlp_tile_logit(w, bias, cur, half);
        if (half == 0 && base + col < n) out[base + col] = sigmoidf_(z);
#pragma unroll
        for (uint32_t st = 0; st < kFeat / 2; ++st) cur[st] = nxt[st];
    }
}

// Gradient: a workgroup of four wavefronts takes groups of 16 samples and runs them
// forward and backward on 16x16 fp32 matrix tiles, wavefront w owning hidden units
// 16 w .. 16 w + 15 of both layers.  In a result tile a lane holds samples 4 g .. 4 g
// + 3 (g = lane / 16) of unit 16 w + lane % 16, so the ReLU masks of the backward
// pass are read from the registers of the forward one; the activations and deltas
// the next product needs as operands go through LDS.  The first layer's bias is its
// 13th input row (x = 1), which gives its gradient with the weights'.  The weight
// gradients stay in registers over the workgroup's groups; each workgroup writes one
// partial gradient, and k_mlp_reduce sums them in a fixed order, so the result does
// not depend on scheduling.
//
// A batch of 1024 samples is 64 workgroups of one group: bound by the chain of five
// products and their barriers, 7.6 us (a sample a lane with the two layers' 5000
// multiply-adds in sequence, 32 lanes of each workgroup busy: 119 us).
__global__ __launch_bounds__(256) void k_mlp_grad(const float *__restrict__ p, const float *__restrict__ x,
                                                  const float *__restrict__ y, const uint32_t *__restrict__ order,
                                                  uint64_t first, uint32_t n, float inv_n, float *__restrict__ partials) {
    // row strides: operand reads take rows lane % 16 (stride 4 mod 64: banks 4 i + g)
    // or rows g (any), and W2 by rows g (stride 16 mod 64: banks 16 g + i)
    constexpr int B = kGradSamples, LW = 80, LH = 68, LX = 20;
    __shared__ float w2[kHid][LW];
    __shared__ float sx[B][LX], sh1[B][LH], sd2[B][LH], sd1[B][LH];
    __shared__ float sz[4][B], sy[B], sdz3[B];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6, i = lane & 15, g = lane >> 4;
    const uint32_t unit = 16 * wave + i;
#pragma unroll
    for (uint32_t k = 0; k < kHid * kHid / 256; ++k) {
        const uint32_t e = t + 256 * k;
        w2[e / kHid][e % kHid] = p[kOffW2 + e];
    }
    float w1[4];  // rows 4 s + g of (W1, b1, 0, 0, 0)
#pragma unroll
    for (uint32_t s = 0; s < 4; ++s) {
        const uint32_t k = 4 * s + g;
        w1[s] = k < (uint32_t)kFeat ? p[kOffW1 + k * kHid + unit] : k == (uint32_t)kFeat ? p[kOffB1 + unit] : 0.f;
    }
    const float b2 = p[kOffB2 + unit], w3 = p[kOffW3 + unit], b3 = p[kOffB3];
    f32x4 gw2[4], gw1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) gw2[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    float gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, gl = 0.f;
    const uint32_t groups = (n + B - 1) / B;
    for (uint32_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
        {  // 16 rows of 12 features, a one and three zeros; a lane of the zeros fetches the label
            const uint32_t r = t >> 4, k = t & 15;
            const uint64_t s = (uint64_t)grp * B + r;
            const bool ok = s < n;
            const uint64_t row = !ok ? 0 : order ? order[first + s] : first + s;
            sx[r][k] = k < (uint32_t)kFeat ? (ok ? x[row * kFeat + k] : 0.f) : k == (uint32_t)kFeat ? 1.f : 0.f;
            if (k == 15) sy[r] = ok ? y[row] : 0.f;
        }
        __syncthreads();
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (uint32_t s = 0; s < 4; ++s) a = __builtin_amdgcn_mfma_f32_16x16x4f32(sx[i][4 * s + g], w1[s], a, 0, 0, 0);
        float h1[4], h2[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            h1[r] = fmaxf(a[r], 0.f);
            sh1[4 * g + r][unit] = h1[r];
        }
        __syncthreads();
        f32x4 c = {b2, b2, b2, b2};
#pragma unroll
        for (uint32_t s = 0; s < kHid / 4; ++s)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(sh1[i][4 * s + g], w2[4 * s + g][unit], c, 0, 0, 0);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            h2[r] = fmaxf(c[r], 0.f);
            float z = h2[r] * w3;  // summed over the wavefront's 16 units
#pragma unroll
            for (uint32_t d = 1; d < 16; d <<= 1) z += __shfl_xor(z, d);
            if (i == 0) sz[wave][4 * g + r] = z;
        }
        __syncthreads();
        if (t < (uint32_t)B) {
            const bool ok = (uint64_t)grp * B + t < n;
            const float z = b3 + ((sz[0][t] + sz[1][t]) + (sz[2][t] + sz[3][t]));
            const float d = ok ? (sigmoidf_(z) - sy[t]) * inv_n : 0.f;
            sdz3[t] = d;
            gb3 += d;
            gl += ok ? bce_logit(z, sy[t]) * inv_n : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const float d3 = sdz3[4 * g + r];
            const float d2 = h2[r] > 0.f ? d3 * w3 : 0.f;
            sd2[4 * g + r][unit] = d2;
            gb2 += d2;
            gw3 = fmaf(d3, h2[r], gw3);
        }
        __syncthreads();
        f32x4 e = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (uint32_t s = 0; s < kHid / 4; ++s)
            e = __builtin_amdgcn_mfma_f32_16x16x4f32(sd2[i][4 * s + g], w2[unit][4 * s + g], e, 0, 0, 0);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) sd1[4 * g + r][unit] = h1[r] > 0.f ? e[r] : 0.f;
#pragma unroll
        for (uint32_t s = 0; s < B / 4; ++s) {  // rows `unit` of W2's gradient, all 64 columns
            const float h = sh1[4 * s + g][unit];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                gw2[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(h, sd2[4 * s + g][16 * q + i], gw2[q], 0, 0, 0);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t s = 0; s < B / 4; ++s)
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sx[4 * s + g][i], sd1[4 * s + g][unit], gw1, 0, 0, 0);
        __syncthreads();  // the next group overwrites sx
    }
    float *out = partials + (uint64_t)blockIdx.x * (kParams + 1);
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t row = 4 * g + r;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) out[kOffW2 + (16 * wave + row) * kHid + 16 * q + i] = gw2[q][r];
        if (row < (uint32_t)kFeat) out[kOffW1 + row * kHid + unit] = gw1[r];
        if (row == (uint32_t)kFeat) out[kOffB1 + unit] = gw1[r];
    }
    gb2 += __shfl_xor(gb2, 16);
    gb2 += __shfl_xor(gb2, 32);
    gw3 += __shfl_xor(gw3, 16);
    gw3 += __shfl_xor(gw3, 32);
    if (g == 0) {
        out[kOffB2 + unit] = gb2;
        out[kOffW3 + unit] = gw3;
    }
#pragma unroll
    for (uint32_t d = 1; d < (uint32_t)B; d <<= 1) {  // lanes 0..15 of wavefront 0 hold the sums
        gb3 += __shfl_xor(gb3, d);
        gl += __shfl_xor(gl, d);
    }
    if (t == 0) {
        out[kOffB3] = gb3;
        out[kParams] = gl;
    }
}

// The sum over rows of partials[row][i], entry kParams the loss: a workgroup takes 64
// entries, its four wavefronts every fourth row, in a fixed order.  ADAM: the entry's
// parameter takes its Adam step at once (a training step is two launches); otherwise
// the sum goes to grad.  64 rows: 3.7 us with the Adam step (one thread summing the
// 32 rows of an entry, a copy of the loss and Adam as launches of their own: 18 us).
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ partials, uint32_t rows,
                                                    float *__restrict__ grad, float *__restrict__ loss,
                                                    float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                                    float lr, float beta1, float beta2, float eps, float c1, float c2) {
    __shared__ float part[4][64];
    const uint32_t c = threadIdx.x & 63, wave = threadIdx.x >> 6, i = blockIdx.x * 64 + c;
    const float *src = partials + min(i, (uint32_t)kParams);
    float a = 0.f;
#pragma unroll 8
    for (uint32_t r = wave; r < rows; r += 4) a += src[(uint64_t)r * (kParams + 1)];
    part[wave][c] = a;
    __syncthreads();
    if (wave != 0 || i > (uint32_t)kParams) return;
    const float gi = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
    if (i == (uint32_t)kParams) {
        *loss = gi;
    } else if (!ADAM) {
        grad[i] = gi;
    } else {
        const float mi = beta1 * m[i] + (1.f - beta1) * gi;
        const float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

MlpWork &mlp_work(Ctx &c) {
    if (!c.mlp) {
        auto w = std::make_unique<MlpWork>();
        w->params = (float *)c.dalloc(kParams * 4);
        w->m = (float *)c.dalloc(kParams * 4);
        w->v = (float *)c.dalloc(kParams * 4);
        w->grad = (float *)c.dalloc(kParams * 4);
        w->loss = (float *)c.dalloc(256);
        GSS_HIP(hipHostMalloc((void **)&w->h_loss, 256, hipHostMallocDefault));
        c.mlp = w.release();
    }
    return *c.mlp;
}

void mlp_release(Ctx &c) {
    MlpWork *w = c.mlp;
    if (!w) return;
    c.dfree(w->params);
    c.dfree(w->m);
    c.dfree(w->v);
    c.dfree(w->grad);
    c.dfree(w->partials);
    c.dfree(w->loss);
    c.dfree(w->stage);
    if (w->h_loss) (void)hipHostFree(w->h_loss);
    delete w;
    c.mlp = nullptr;
}

char *mlp_stage(Ctx &c, MlpWork &w, size_t bytes) {
    if (bytes > w.stage_bytes) {
        c.sync();  // queued work may still read the old buffer
        c.dfree(w.stage);
        w.stage = nullptr;
        w.stage_bytes = 0;
        const size_t want = std::max<size_t>(bytes, (size_t)1 << 20);
        w.stage = (char *)c.dalloc(want);
        w.stage_bytes = want;
    }
    return w.stage;
}

// Queues the partial gradients; returns their number.
static uint32_t queue_partials(Ctx &c, MlpWork &w, const float *x, const float *y, const uint32_t *order, uint64_t first,
                               uint32_t n) {
    const uint32_t blocks = std::min<uint32_t>((n + kGradSamples - 1) / kGradSamples, kGradBlocks);
    if (blocks > w.partial_rows) {
        c.sync();
        c.dfree(w.partials);
        w.partials = nullptr;
        w.partial_rows = 0;
        const uint32_t rows = std::max<uint32_t>(blocks, 64);
        w.partials = (float *)c.dalloc((size_t)rows * (kParams + 1) * 4);
        w.partial_rows = rows;
    }
    hipLaunchKernelGGL(k_mlp_grad, dim3(blocks), dim3(256), 0, c.stream, w.params, x, y, order, first, n, 1.f / n,
                       w.partials);
    GSS_HIP(hipGetLastError());
    return blocks;
}

constexpr unsigned kReduceBlocks = (kParams + 1 + 63) / 64;

void mlp_queue_grad(Ctx &c, MlpWork &w, const float *x, const float *y, const uint32_t *order, uint64_t first,
                    uint32_t n) {
    const uint32_t rows = queue_partials(c, w, x, y, order, first, n);
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(kReduceBlocks), dim3(256), 0, c.stream, w.partials, rows, w.grad, w.loss,
                       nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
    GSS_HIP(hipGetLastError());
}

void mlp_queue_step(Ctx &c, MlpWork &w, const float *x, const float *y, const uint32_t *order, uint64_t first,
                    uint32_t n, float lr, float beta1, float beta2, float eps, float *loss) {
    w.step++;
    const double c1 = 1.0 - std::pow((double)beta1, (double)w.step);
    const double c2 = 1.0 - std::pow((double)beta2, (double)w.step);
    const uint32_t rows = queue_partials(c, w, x, y, order, first, n);
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(kReduceBlocks), dim3(256), 0, c.stream, w.partials, rows, nullptr, loss,
                       w.params, w.m, w.v, lr, beta1, beta2, eps, (float)c1, (float)c2);
    GSS_HIP(hipGetLastError());
}

unsigned mlp_grid(const Ctx &c, uint64_t n) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + 127) / 128, (uint64_t)c.n_cu * 2));
}

// Queues the upload of host parameters into w.params through the upload ring.
static void upload_params(Ctx &c, MlpWork &w, const float *params) {
    const Ctx::Staged st = c.stage_upload(kParams * 4);
    std::memcpy(st.h, params, kParams * 4);
    GSS_HIP(hipMemcpyAsync(w.params, st.h, kParams * 4, hipMemcpyHostToDevice, c.stream));
    c.stage_done(st);
}

// A device view of an input array (host arrays are copied to the stage at `off`).
static const char *device_input(Ctx &c, char *stage, size_t off, const void *p, size_t bytes) {
    if (is_device_pointer(p)) return (const char *)p;
    GSS_HIP(hipMemcpyAsync(stage + off, p, bytes, hipMemcpyHostToDevice, c.stream));
    return stage + off;
}

static size_t round256(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace gss

using namespace gss;

extern "C" gss_status gss_mlp_forward(gss_ctx *ctx, const float *params, const float *x, uint32_t n, float *out) {
    GSS_API_BEGIN(ctx)
    Ctx &c = *c_;
    GSS_REQUIRE(params && x && out, GSS_ERR_INVALID_ARG, "null argument");
    if (n == 0) return GSS_OK;
    GSS_REQUIRE(!c.pending, GSS_ERR_STATE, "a test is in flight");
    MlpWork &w = mlp_work(c);
    upload_params(c, w, params);
    const size_t xb = round256((size_t)n * kFeat * 4), ob = round256((size_t)n * 4);
    c.sync();  // the stage may be replaced: nothing queued reads it
    char *st = mlp_stage(c, w, xb + ob);
    const float *dx = (const float *)device_input(c, st, 0, x, (size_t)n * kFeat * 4);
    const bool dev_out = is_device_pointer(out);
    float *dout = dev_out ? out : (float *)(st + xb);
    hipLaunchKernelGGL(k_mlp_forward, dim3(mlp_grid(c, n)), dim3(256), 0, c.stream, w.params, dx, n, dout);
    GSS_HIP(hipGetLastError());
    if (!dev_out) GSS_HIP(hipMemcpyAsync(out, dout, (size_t)n * 4, hipMemcpyDeviceToHost, c.stream));
    c.sync();
    GSS_API_END
}

extern "C" gss_status gss_mlp_loss_grad(gss_ctx *ctx, const float *params, const float *x, const float *y, uint32_t n,
                                        float *out_loss, float *out_grad) {
    GSS_API_BEGIN(ctx)
    Ctx &c = *c_;
    GSS_REQUIRE(params && x && y && out_loss && out_grad, GSS_ERR_INVALID_ARG, "null argument");
    GSS_REQUIRE(n >= 1, GSS_ERR_INVALID_ARG, "n must be at least 1");
    GSS_REQUIRE(!c.pending, GSS_ERR_STATE, "a test is in flight");
    MlpWork &w = mlp_work(c);
    upload_params(c, w, params);
    const size_t xb = round256((size_t)n * kFeat * 4), yb = round256((size_t)n * 4);
    c.sync();
    char *st = mlp_stage(c, w, xb + yb);
    const float *dx = (const float *)device_input(c, st, 0, x, (size_t)n * kFeat * 4);
    const float *dy = (const float *)device_input(c, st, xb, y, (size_t)n * 4);
    mlp_queue_grad(c, w, dx, dy, nullptr, 0, n);
    GSS_HIP(hipMemcpyAsync(w.h_loss, w.loss, 4, hipMemcpyDeviceToHost, c.stream));
    GSS_HIP(hipMemcpyAsync(out_grad, w.grad, kParams * 4,
                           is_device_pointer(out_grad) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c.stream));
    c.sync();
    *out_loss = *w.h_loss;
    GSS_API_END
}

extern "C" gss_status gss_mlp_train(gss_ctx *ctx, float *params, const float *x, const float *y, uint32_t n,
                                    const uint32_t *order, uint64_t n_order, const gss_adam_config *cfg,
                                    float *out_losses) {
    GSS_API_BEGIN(ctx)
    Ctx &c = *c_;
    GSS_REQUIRE(params && x && y && order && cfg, GSS_ERR_INVALID_ARG, "null argument");
    GSS_REQUIRE(n >= 1 && n_order >= 1, GSS_ERR_INVALID_ARG, "n and n_order must be at least 1");
    GSS_REQUIRE(cfg->batch >= 1, GSS_ERR_INVALID_ARG, "batch must be at least 1");
    GSS_REQUIRE(cfg->lr > 0 && cfg->beta1 >= 0 && cfg->beta1 < 1 && cfg->beta2 >= 0 && cfg->beta2 < 1 && cfg->eps > 0,
                GSS_ERR_INVALID_ARG, "Adam settings out of range");
    GSS_REQUIRE(!is_device_pointer(order), GSS_ERR_INVALID_ARG, "order must be a host array");
    for (uint64_t i = 0; i < n_order; ++i)
        GSS_REQUIRE(order[i] < n, GSS_ERR_INVALID_ARG, "order entry beyond n");
    GSS_REQUIRE(!c.pending, GSS_ERR_STATE, "a test is in flight");
    MlpWork &w = mlp_work(c);
    upload_params(c, w, params);
    launch_fill_u32(c, (uint32_t *)w.m, kParams, 0);
    launch_fill_u32(c, (uint32_t *)w.v, kParams, 0);
    w.step = 0;
    const uint64_t steps = (n_order + cfg->batch - 1) / cfg->batch;
    const size_t xb = round256((size_t)n * kFeat * 4), yb = round256((size_t)n * 4), ob = round256(n_order * 4),
                 lb = round256(steps * 4);
    c.sync();
    char *st = mlp_stage(c, w, xb + yb + ob + lb);
    const float *dx = (const float *)device_input(c, st, 0, x, (size_t)n * kFeat * 4);
    const float *dy = (const float *)device_input(c, st, xb, y, (size_t)n * 4);
    GSS_HIP(hipMemcpyAsync(st + xb + yb, order, n_order * 4, hipMemcpyHostToDevice, c.stream));
    const uint32_t *dorder = (const uint32_t *)(st + xb + yb);
    float *dlosses = (float *)(st + xb + yb + ob);
    for (uint64_t k = 0; k < steps; ++k) {
        const uint64_t first = k * cfg->batch;
        const uint32_t nb = (uint32_t)std::min<uint64_t>(cfg->batch, n_order - first);
        mlp_queue_step(c, w, dx, dy, dorder, first, nb, cfg->lr, cfg->beta1, cfg->beta2, cfg->eps, dlosses + k);
    }
    GSS_HIP(hipMemcpyAsync(params, w.params, kParams * 4, hipMemcpyDeviceToHost, c.stream));
    if (out_losses) GSS_HIP(hipMemcpyAsync(out_losses, dlosses, steps * 4, hipMemcpyDeviceToHost, c.stream));
    c.sync();
    GSS_API_END
}
