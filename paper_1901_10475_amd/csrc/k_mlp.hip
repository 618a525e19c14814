// k_mlp.hip -- the per-object step network: features, BF16 inference, FP32
// training (forward, backward, Adam) and the per-object record counts that the
// training targets are built from.
//
// The paper keeps a time interval per object so that objects far from all
// others take long intervals (Sec. Collision Detection with 4D AABB Trees;
// Procedure advanceTime) but leaves the choice of step open.  This network
// predicts log2(step in seconds) from five orbital features:
//   x = (a / 42164, e, i / pi, r_p / 42164, vmax / 8),  r_p = a (1 - e),
//   h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2), y = w3 . h2 + b3,
//   step = clamp(floor(2^y / tick), 1, max(T, 1)) ticks.
// Any step keeps the boxes conservative, so the network changes cost only.
//
// Inference runs one object per lane: BF16 weights staged in LDS (read as
// wave-uniform broadcasts), BF16 inputs and hidden activations packed two to a
// register, FP32 accumulation through v_dot2c_f32_bf16.  Training keeps FP32
// master weights: one kernel runs the forward and backward pass and sums the
// gradients of its samples, on the FP32 matrix instructions; a second adds the
// partial gradients in a fixed order, so gradients are deterministic.
#include "cd_internal.h"

namespace cd {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// FP32 -> bfloat16 bits, round to nearest, ties to even.
__device__ inline uint32_t bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if (f != f)
        return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ inline float bf16_value(uint32_t h) { return __uint_as_float(h << 16); }

__device__ inline float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a),
                                           __builtin_bit_cast(bf16x2, b), c, false);
}

__device__ inline void mlp_features(double a, double e, double inc, double mu, double x[5],
                                    double &vmax)
{
    double rp = a * (1.0 - e);
    vmax = sqrt(mu * (1.0 + e) / rp);
    x[0] = a / 42164.0;
    x[1] = e;
    x[2] = inc / 3.141592653589793;
    x[3] = rp / 42164.0;
    x[4] = vmax / 8.0;
}

__global__ void k_mlp_features(cd_elements el, double mu, float *xo)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= el.n)
        return;
    double x[5], vmax;
    mlp_features(el.a[i], el.e[i], el.inc[i], mu, x, vmax);
    for (int f = 0; f < kMlpIn; ++f)
        xo[i * kMlpIn + f] = (float)x[f];
}

// ---- BF16 inference -----------------------------------------------------------------

__global__ __launch_bounds__(256) void k_dt_mlp(cd_elements el, const uint16_t *__restrict__ w,
                                                double mu, double tick_s, double fallback,
                                                uint32_t T, uint32_t *dt, float *yout)
{
    __shared__ uint4 sW2[kMlpHid][8];     // row r: bf16 pairs (2k, 2k+1), k < 32
    __shared__ uint32_t sW1[kMlpHid][3];  // row r: pairs (x0 x1), (x2 x3), (x4 0)
    __shared__ float sB1[kMlpHid], sB2[kMlpHid], sW3[kMlpHid];
    __shared__ float sB3;
    uint32_t *w2 = (uint32_t *)&sW2[0][0];
    for (int t = threadIdx.x; t < kMlpHid * 32; t += blockDim.x) {
        int r = t >> 5, k = t & 31;
        const uint16_t *row = w + kMlpW2 + r * kMlpHid;
        w2[t] = (uint32_t)row[2 * k] | ((uint32_t)row[2 * k + 1] << 16);
    }
    for (int t = threadIdx.x; t < kMlpHid * 3; t += blockDim.x) {
        int r = t / 3, q = t % 3;
        const uint16_t *row = w + kMlpW1 + r * kMlpIn;
        uint32_t lo = row[2 * q];
        uint32_t hi = (2 * q + 1 < kMlpIn) ? (uint32_t)row[2 * q + 1] : 0u;
        sW1[r][q] = lo | (hi << 16);
    }
    for (int t = threadIdx.x; t < kMlpHid; t += blockDim.x) {
        sB1[t] = bf16_value(w[kMlpB1 + t]);
        sB2[t] = bf16_value(w[kMlpB2 + t]);
        sW3[t] = bf16_value(w[kMlpW3 + t]);
    }
    if (threadIdx.x == 0)
        sB3 = bf16_value(w[kMlpB3]);
    __syncthreads();

    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= el.n)
        return;
    double xd[5], vmax;
    mlp_features(el.a[i], el.e[i], el.inc[i], mu, xd, vmax);
    uint32_t xb[5];
    for (int f = 0; f < 5; ++f)
        xb[f] = bf16_bits((float)xd[f]);
    uint32_t x01 = xb[0] | (xb[1] << 16), x23 = xb[2] | (xb[3] << 16), x4 = xb[4];

    uint32_t h1[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        uint32_t hb[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int r = 2 * k + q;
            float acc = sB1[r];
            acc = dot2_bf16(sW1[r][0], x01, acc);
            acc = dot2_bf16(sW1[r][1], x23, acc);
            acc = dot2_bf16(sW1[r][2], x4, acc);
            hb[q] = bf16_bits(fmaxf(acc, 0.0f));
        }
        h1[k] = hb[0] | (hb[1] << 16);
    }
    float y = 0.0f;
    for (int r = 0; r < kMlpHid; ++r) {
        float acc = sB2[r];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            uint4 wv = sW2[r][q];
            acc = dot2_bf16(wv.x, h1[4 * q + 0], acc);
            acc = dot2_bf16(wv.y, h1[4 * q + 1], acc);
            acc = dot2_bf16(wv.z, h1[4 * q + 2], acc);
            acc = dot2_bf16(wv.w, h1[4 * q + 3], acc);
        }
        float h2 = bf16_value(bf16_bits(fmaxf(acc, 0.0f)));
        y = fmaf(sW3[r], h2, y);
    }
    y += sB3;
    if (yout)
        yout[i] = y;
    uint32_t d;
    if (isfinite(y)) {
        double v = floor(exp2((double)y) / tick_s);
        double cap = T > 0 ? (double)T : 1.0;
        v = v < 1.0 ? 1.0 : (v > cap ? cap : v);
        d = (uint32_t)v;
    } else {
        d = heuristic_step(vmax, tick_s, fallback, T);
    }
    dt[i] = d;
}

// ---- FP32 training ----------------------------------------------------------------------

struct MlpF32 {
    float W1[kMlpHid][kMlpIn];
    float b1[kMlpHid];
    float4 W2[kMlpHid][kMlpHid / 4];
    float b2[kMlpHid];
    float w3[kMlpHid];
    float b3;
};

__device__ inline void load_mlp_f32(MlpF32 &s, const float *__restrict__ w)
{
    float *W1 = &s.W1[0][0];
    float *W2 = (float *)&s.W2[0][0];
    for (int t = threadIdx.x; t < kMlpHid * kMlpHid; t += blockDim.x)
        W2[t] = w[kMlpW2 + t];
    for (int t = threadIdx.x; t < kMlpHid * kMlpIn; t += blockDim.x)
        W1[t] = w[kMlpW1 + t];
    for (int t = threadIdx.x; t < kMlpHid; t += blockDim.x) {
        s.b1[t] = w[kMlpB1 + t];
        s.b2[t] = w[kMlpB2 + t];
        s.w3[t] = w[kMlpW3 + t];
    }
    if (threadIdx.x == 0)
        s.b3 = w[kMlpB3];
    __syncthreads();
}

__device__ inline void mlp_layer1(const MlpF32 &s, const float x[5], float h1[kMlpHid])
{
#pragma unroll
    for (int r = 0; r < kMlpHid; ++r) {
        float acc = s.b1[r];
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c)
            acc = fmaf(s.W1[r][c], x[c], acc);
        h1[r] = fmaxf(acc, 0.0f);
    }
}

__device__ inline float mlp_row2(const MlpF32 &s, int r, const float h1[kMlpHid])
{
    float acc = s.b2[r];
#pragma unroll
    for (int q = 0; q < kMlpHid / 4; ++q) {
        float4 wv = s.W2[r][q];
        acc = fmaf(wv.x, h1[4 * q + 0], acc);
        acc = fmaf(wv.y, h1[4 * q + 1], acc);
        acc = fmaf(wv.z, h1[4 * q + 2], acc);
        acc = fmaf(wv.w, h1[4 * q + 3], acc);
    }
    return acc;
}

__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ w,
                                                     const float *__restrict__ x, uint32_t B,
                                                     float *__restrict__ y)
{
    __shared__ MlpF32 s;
    load_mlp_f32(s, w);
    uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B)
        return;
    float xv[kMlpIn], h1[kMlpHid];
    for (int c = 0; c < kMlpIn; ++c)
        xv[c] = x[(uint64_t)b * kMlpIn + c];
    mlp_layer1(s, xv, h1);
    float out = s.b3;
#pragma unroll 1
    for (int r = 0; r < kMlpHid; ++r)
        out = fmaf(s.w3[r], fmaxf(mlp_row2(s, r, h1), 0.0f), out);
    y[b] = out;
}

// Gradients: forward and backward pass and the per-parameter sums in one kernel,
// 64 samples (a tile) at a time, activations and their gradients in LDS.  The
// three 64 x 64 x 64 products of a tile -- z2 = h1 W2^T, dh1 = dz2 W2 and
// gW2 = dz2^T h1 -- run on the FP32 matrix instructions (32 x 32 x 2, one
// quadrant a wave; gW2 accumulates in registers over the workgroup's tiles), the
// small sums on the lanes.  Rows of 65 words: lanes along a row and along a
// column both meet different banks.
// Bound: latency; a workgroup alone takes 12 us for a tile, 2.6 of them matrix
// instructions, so up to three share a CU.  33 696 samples: 24 us, and 4 for the
// sum of the partials (264 workgroups of two tiles 27); a kernel that kept 258
// rows of activations in memory and another for their outer products by scalar
// FMA took 145, the serial sum of 264 partials 63.  Relative error of the gradient
// against 64 bits, six batches each, before and now: 64 samples 9.9e-8 and 7.2e-8,
// 1 000 7.7e-8 and 6.4e-8, 16 848 1.4e-7 and 6.4e-8, 33 696 2.1e-7 and 6.3e-8 (of
// the loss, a single sum that now and then rounds the other way, 6.2e-8 and 4.1e-8,
// 9.5e-8 and 7.0e-8, 5.9e-8 and 6.3e-8, 2.5e-7 and 6.2e-8).
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kGradTile = 64, kGradRow = 65, kGradThreads = 256, kGradWaves = kGradThreads / 64,
              kGradSpan = kGradTile / kGradWaves;   // samples (or terms) of a wave
// Workgroups, and so partial gradients, at most (three on a CU), with equal
// numbers of tiles.
uint32_t mlp_grad_blocks(uint32_t B)
{
    constexpr uint32_t kMost = 768;
    const uint32_t tiles = (uint32_t)(((uint64_t)B + kGradTile - 1) / kGradTile),
                   each = (tiles + kMost - 1) / kMost;
    return tiles ? (tiles + each - 1) / each : 0u;
}

// acc += A B for one wave's 32 x 32 quadrant and 64 terms: a(m, k) and b(k, n)
// are read for m, n = lane % 32 and k = 2 step + lane / 32; acc[4 i + j] is row
// 8 i + 4 (lane / 32) + j, column lane % 32.
template <class A, class B>
__device__ inline f32x16 quadrant(f32x16 acc, A &&a, B &&b)
{
#pragma unroll 8
    for (int step = 0; step < 32; ++step)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a(step), b(step), acc, 0, 0, 0);
    return acc;
}

__global__ __launch_bounds__(kGradThreads)
__attribute__((amdgpu_waves_per_eu(3))) void k_mlp_grad(const float *__restrict__ w,
                                                           const float *__restrict__ x,
                                                           const float *__restrict__ target,
                                                           uint32_t B, float *__restrict__ part)
{
    // h2: relu(z2), then dz2, then dz1
    __shared__ float h1[kGradTile * kGradRow], h2[kGradTile * kGradRow],
        w2[kMlpHid * kGradRow];
    __shared__ float xs[kGradTile][kMlpIn], sw3[kMlpHid], ypart[kGradWaves][kGradTile],
        dys[kGradTile];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 31, half = lane >> 5, qm = (wv >> 1) * 32, qn = (wv & 1) * 32;
    float w1[kMlpIn];
    for (int k = threadIdx.x; k < kMlpHid * kMlpHid; k += kGradThreads)
        w2[k / kMlpHid * kGradRow + k % kMlpHid] = w[kMlpW2 + k];
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c)
        w1[c] = w[kMlpW1 + lane * kMlpIn + c];
    const float b1 = w[kMlpB1 + lane], b2 = w[kMlpB2 + qn + col], w3 = w[kMlpW3 + lane],
                b3 = w[kMlpB3];
    if (wv == 0)
        sw3[lane] = w3;
    f32x16 g2 = {};
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f, gw1[kMlpIn] = {};
    const uint32_t tiles = (uint32_t)(((uint64_t)B + kGradTile - 1) / kGradTile);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t s0 = tile * kGradTile, n = B - s0 < kGradTile ? B - s0 : kGradTile;
        const int first = wv * kGradSpan;   // this wave's samples where lanes are units
        __syncthreads();   // the last tile's LDS has been read
        for (int k = threadIdx.x; k < kGradTile * kMlpIn; k += kGradThreads)
            xs[k / kMlpIn][k % kMlpIn] =
                (uint32_t)(k / kMlpIn) < n ? x[(uint64_t)s0 * kMlpIn + k] : 0.0f;
        const float want = target[s0 + ((uint32_t)lane < n ? lane : n - 1)];
        __syncthreads();
#pragma unroll 4
        for (int q = 0; q < kGradSpan; ++q) {
            float acc = b1;
#pragma unroll
            for (int c = 0; c < kMlpIn; ++c)
                acc = fmaf(w1[c], xs[first + q][c], acc);
            // samples past the batch: no activation, no gradient
            h1[(first + q) * kGradRow + lane] = (uint32_t)(first + q) < n ? fmaxf(acc, 0.0f) : 0.0f;
        }
        __syncthreads();
        {
            f32x16 z;
#pragma unroll
            for (int k = 0; k < 16; ++k)
                z[k] = b2;
            z = quadrant(
                z, [&](int k) { return h1[(qm + col) * kGradRow + 2 * k + half]; },
                [&](int k) { return w2[(qn + col) * kGradRow + 2 * k + half]; });
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int s = qm + 8 * (k / 4) + 4 * half + k % 4;
                h2[s * kGradRow + qn + col] = (uint32_t)s < n ? fmaxf(z[k], 0.0f) : 0.0f;
            }
        }
        __syncthreads();
        {   // y, lanes along the samples, each wave a quarter of the units
            float y = 0.0f;
#pragma unroll
            for (int q = 0; q < kGradSpan; ++q)
                y = fmaf(sw3[first + q], h2[lane * kGradRow + first + q], y);
            ypart[wv][lane] = y;
        }
        __syncthreads();
        {
            float y = b3;
#pragma unroll
            for (int q = 0; q < kGradWaves; ++q)
                y += ypart[q][lane];
            const float res = (uint32_t)lane < n ? y - want : 0.0f, dy = 2.0f * res / (float)B;
            gb3 += dy;
            loss += res * res / (float)B;
            if (wv == 0)
                dys[lane] = dy;
        }
        __syncthreads();
#pragma unroll 4
        for (int q = 0; q < kGradSpan; ++q) {
            float &at = h2[(first + q) * kGradRow + lane];
            const float h = at, dy = dys[first + q], dz = h > 0.0f ? dy * w3 : 0.0f;
            gw3 = fmaf(dy, h, gw3);
            gb2 += dz;
            at = dz;
        }
        __syncthreads();
        f32x16 dh = {};
        dh = quadrant(
            dh, [&](int k) { return h2[(qm + col) * kGradRow + 2 * k + half]; },
            [&](int k) { return w2[(2 * k + half) * kGradRow + qn + col]; });
        g2 = quadrant(
            g2, [&](int k) { return h2[(2 * k + half) * kGradRow + qm + col]; },
            [&](int k) { return h1[(2 * k + half) * kGradRow + qn + col]; });
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int at = (qm + 8 * (k / 4) + 4 * half + k % 4) * kGradRow + qn + col;
            h2[at] = h1[at] > 0.0f ? dh[k] : 0.0f;
        }
        __syncthreads();
#pragma unroll 4
        for (int q = 0; q < kGradSpan; ++q) {
            const float dz = h2[(first + q) * kGradRow + lane];
            gb1 += dz;
#pragma unroll
            for (int c = 0; c < kMlpIn; ++c)
                gw1[c] = fmaf(dz, xs[first + q][c], gw1[c]);
        }
    }
    // the workgroup's partial gradient
    float *const out = part + (uint64_t)blockIdx.x * (kMlpParams + 1);
#pragma unroll
    for (int k = 0; k < 16; ++k)
        out[kMlpW2 + (qm + 8 * (k / 4) + 4 * half + k % 4) * kMlpHid + qn + col] = g2[k];
    constexpr int kSmall = 3 + kMlpIn;   // per unit: gb1, gb2, gw3, gW1
    __syncthreads();
    {
        float *const red = h1 + (wv * kSmall) * 64 + lane;
        red[0] = gb1;
        red[64] = gb2;
        red[128] = gw3;
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c)
            red[(3 + c) * 64] = gw1[c];
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kSmall * 64; k += kGradThreads) {
        float sum = 0.0f;
        for (int q = 0; q < kGradWaves; ++q)
            sum += h1[q * kSmall * 64 + k];
        const int f = k / 64, u = k % 64;
        out[f == 0 ? kMlpB1 + u : f == 1 ? kMlpB2 + u : f == 2 ? kMlpW3 + u
                                                               : kMlpW1 + u * kMlpIn + f - 3] = sum;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        gb3 += __shfl_xor(gb3, o, 64);
        loss += __shfl_xor(loss, o, 64);
    }
    if (threadIdx.x == 0) {
        out[kMlpB3] = gb3;
        out[kMlpParams] = loss;
    }
}

// Gradient entry = sum of the partials, kReduceSlices strided sums of them added
// in order (the same every time).
constexpr int kReduceSlices = 16;

__global__ __launch_bounds__(64 * kReduceSlices) void k_mlp_reduce(const float *__restrict__ part,
                                                                   uint32_t nblk,
                                                                   float *__restrict__ grad,
                                                                   float *__restrict__ loss)
{
    __shared__ float red[kReduceSlices][64];
    const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    float sum = 0.0f;
    if (p <= kMlpParams) {
#pragma unroll 8
        for (uint32_t k = slice; k < nblk; k += kReduceSlices)
            sum += part[(uint64_t)k * (kMlpParams + 1) + p];
    }
    red[slice][lane] = sum;
    __syncthreads();
    if (slice != 0 || p > kMlpParams)
        return;
#pragma unroll
    for (int q = 1; q < kReduceSlices; ++q)
        sum += red[q][lane];
    if (p < kMlpParams)
        grad[p] = sum;
    else if (loss)
        *loss = sum;
}

// Adam (Kingma & Ba) with bias-corrected moments; optional BF16 export.
__global__ void k_mlp_adam(float *w, float *m, float *v, const float *g, int64_t step, float lr,
                           float beta1, float beta2, float eps, uint16_t *wb)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kMlpParams)
        return;
    float gp = g[p];
    float mp = beta1 * m[p] + (1.0f - beta1) * gp;
    float vp = beta2 * v[p] + (1.0f - beta2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    float bc1 = (float)(1.0 - pow((double)beta1, (double)step));
    float bc2 = (float)(1.0 - pow((double)beta2, (double)step));
    float wp = w[p] - lr * (mp / bc1) / (sqrtf(vp / bc2) + eps);
    w[p] = wp;
    if (wb)
        wb[p] = (uint16_t)bf16_bits(wp);
}

// Records per object: each record counts once for i and once for j.
__global__ void k_pair_object_counts(const cd_pair *pairs, uint64_t count, uint32_t n,
                                     uint32_t *counts)
{
    uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= count)
        return;
    cd_pair p = pairs[r];
    if (p.i < n)
        atomicAdd(&counts[p.i], 1u);
    if (p.j < n)
        atomicAdd(&counts[p.j], 1u);
}

static inline unsigned blocks_for(uint64_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

hipError_t launch_mlp_features(const cd_elements &el, double mu, float *x, hipStream_t s)
{
    if (el.n == 0)
        return hipSuccess;
    k_mlp_features<<<blocks_for(el.n, 256), 256, 0, s>>>(el, mu, x);
    return hipGetLastError();
}

hipError_t launch_dt_mlp(const cd_elements &el, const uint16_t *w, double mu, double tick_s,
                         double fallback_disp, uint32_t T, uint32_t *dt, float *y,
                         hipStream_t s)
{
    if (el.n == 0)
        return hipSuccess;
    k_dt_mlp<<<blocks_for(el.n, 256), 256, 0, s>>>(el, w, mu, tick_s, fallback_disp, T, dt, y);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *w, const float *x, uint32_t B, float *y,
                              hipStream_t s)
{
    if (B == 0)
        return hipSuccess;
    k_mlp_forward<<<blocks_for(B, 256), 256, 0, s>>>(w, x, B, y);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const float *w, const float *x, const float *target, uint32_t B,
                           float *part, float *grad, float *loss, hipStream_t s)
{
    const uint32_t nblk = mlp_grad_blocks(B);
    k_mlp_grad<<<nblk, kGradThreads, 0, s>>>(w, x, target, B, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    k_mlp_reduce<<<blocks_for(kMlpParams + 1, 64), 64 * kReduceSlices, 0, s>>>(part, nblk, grad,
                                                                               loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *w, float *m, float *v, const float *g, int64_t step,
                           float lr, float beta1, float beta2, float eps, uint16_t *w_bf16,
                           hipStream_t s)
{
    k_mlp_adam<<<blocks_for(kMlpParams, 256), 256, 0, s>>>(w, m, v, g, step, lr, beta1, beta2,
                                                           eps, w_bf16);
    return hipGetLastError();
}

hipError_t launch_pair_object_counts(const cd_pair *pairs, uint64_t count, uint32_t n,
                                     uint32_t *counts, hipStream_t s)
{
    hipError_t e = launch_fill_u32(counts, 0u, n, s);
    if (e != hipSuccess || count == 0)
        return e;
    k_pair_object_counts<<<blocks_for(count, 256), 256, 0, s>>>(pairs, count, n, counts);
    return hipGetLastError();
}

} // namespace cd
