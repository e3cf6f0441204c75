// mlp_train.hip -- training kernels of the learned closure network and the
// standalone forward evaluation.
//
// Loss over a minibatch of n samples: L = (1/n) sum_s ((softplus(o_s) - t_s)
// * inv_scale)^2, o = network output for the sample's raw features (see
// mlp.hpp for the network).  The GEMM operands (weights, x, h1, h2) are rounded
// to bf16 exactly where the sweep's forward rounds them; the rounding has the
// straight-through gradient, and the gradients themselves keep FP32 precision.
// Parameter gradients are summed per workgroup in a fixed order, then over
// workgroups in a fixed order (deterministic).  Adam keeps FP32 master weights; mean / inv_std are not
// trained.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "mlp.hpp"
#include "wlb_internal.hpp"

namespace wlb {

constexpr int kIn = 7, kH = 32;
constexpr int kOffMean = 0, kOffIstd = 7, kOffW1 = 14, kOffB1 = kOffW1 + kH * kIn, kOffW2 = kOffB1 + kH,
              kOffB2 = kOffW2 + kH * kH, kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH, kNParam = kOffB3 + 1;
static_assert(kNParam == 1359, "parameter count");
// GELU and its slope at z, from one evaluation of the CDF's parts.
__device__ __forceinline__ void gelu_and_slope(float z, float &g, float &slope)
{
    const HalfErfc h = half_erfc_parts(z);
    g = fmaf(-(fabsf(z) * h.t), h.e, fmaxf(z, 0.f));
    const float tail = h.t * h.e;
    slope = (z >= 0.f ? 1.0f - tail : tail) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}
__device__ __forceinline__ float sigmoid_f(float o) { return 1.0f / (1.0f + expf(-o)); }

// x as the sum of three bf16 values (8 + 8 + 8 significand bits: nothing of
// an FP32 value is lost; the differences are exact).  A value that bf16
// rounds to infinity keeps it in the first part alone.
struct Split3 {
    __bf16 p[3];
};
__device__ __forceinline__ Split3 split3(float x)
{
    Split3 r;
    r.p[0] = (__bf16)x;
    float d = x - (float)r.p[0];
    d = fabsf(x) < 3e38f ? d : 0.f;
    r.p[1] = (__bf16)d;
    r.p[2] = (__bf16)(d - (float)r.p[1]);
    return r;
}

// Whether an FP32 activation lies within 8 units in the last place of a bf16
// rounding boundary: its FP32 error (some 3e-7 relative) may then put it on
// the other side, which changes the bf16 operand by 2^-8.
__device__ __forceinline__ bool near_boundary(float g)
{
    return ((__float_as_uint(g) & 0xffffu) - (0x8000u - 8u)) <= 16u;
}
// GELU in FP64 to 1.5e-9, rounded to bf16 through FP32.  erfc(u) = t
// exp(-u^2 + P(2 t - 1)), t = 1 / (1 + u / 2), the form that half_erfc_parts
// uses, with P the degree-13 Chebyshev interpolant of log(erfc(u) exp(u^2) / t)
// on 0 < t <= 1 (largest deviation 1.2e-9); exp by 2^k times the Taylor sum of
// the remainder to degree 8 (2e-10).
__device__ __noinline__ __bf16 gelu_bf16(double z)
{
    const double u = fabs(z) * 0.70710678118654752440;
    const double t = 1.0 / fma(0.5, u, 1.0), s = fma(2.0, t, -1.0);
    constexpr double c[14] = {-0.6717940851517218,     0.6726432205460087,      0.04734341752106161,
                              -0.046895482161005086,   -0.0098745349182224,     0.008823558177735913,
                              0.001770666118369054,    -0.002339277724317185,   -0.00018278214127144218,
                              0.0006579538480657341,   -3.211377267356806e-05,  -0.0001546337909289383,
                              1.3371503605768667e-05,  2.0723070945002116e-05};
    double p = c[13];
#pragma unroll
    for (int k = 12; k >= 0; --k) p = fma(p, s, c[k]);
    const double x = fmax(fma(-u, u, p), -700.0);
    const double k = rint(x * 1.4426950408889634);
    const double r = fma(-k, 0.6931471805599453, x);
    double e = 1.0 / 40320.0;
    e = fma(e, r, 1.0 / 5040.0);
    e = fma(e, r, 1.0 / 720.0);
    e = fma(e, r, 1.0 / 120.0);
    e = fma(e, r, 1.0 / 24.0);
    e = fma(e, r, 1.0 / 6.0);
    e = fma(e, r, 0.5);
    e = fma(e, r, 1.0);
    e = fma(e, r, 1.0);
    const double tail = z * (0.5 * t * ldexp(e, (int)k));  // z Phi(-|z|)
    return (__bf16)(float)(z >= 0.0 ? z - tail : tail);
}

constexpr int kGradWG = 512;        // eight wavefronts, each one tile of 32 samples at a time
constexpr int kGradWaves = kGradWG / 64;
constexpr int kTileS = 32;          // samples of a wavefront's tile
constexpr int kMaxGradWG = 512;     // partial rows; larger minibatches loop
constexpr int kRow = kTileS + 8;    // bf16 per LDS row: 16-byte aligned 8-sample reads, rows spread over the banks
// LDS rows of a wavefront's tile, each one quantity of its 32 samples
constexpr int kRowG = 0, kRowH1 = 96, kRowH2 = 128, kRowX = 160, kRowGo = 168, kRows = 171;

typedef __bf16 bf16row_t[kRow];

// Eight consecutive samples of a row as a matrix operand.
__device__ __forceinline__ bf16x8_t row8(const bf16row_t &r, int s) { return *reinterpret_cast<const bf16x8_t *>(&r[s]); }

// Forward and backward pass of the network over a minibatch on the matrix
// cores; per-workgroup gradient partials [gridDim.x][kNParam + 1] (last
// entry: sum of squared residuals).
//
// A wavefront takes 32 samples.  Forward (mlp.hpp's layout): lane l holds the
// sample l % 32 and, in its result registers j, the hidden units mlp_unit(j,
// l / 32); one layer's registers are the next product's operand.  The same
// holds for the backward product with W2^T, whose other operand is FP32: it
// enters as three bf16 parts (split3), three products instead of one, so
// nothing of its 24 bits is lost.  The weight gradients contract over the
// samples: both operands are turned through LDS (rows of one quantity, 32
// samples) and summed over all of a wavefront's tiles in the accumulators of
// dW2 = gz2^T h1, dW1 and db1 = gz1^T [x | 1], db2 = gz2^T [x | 1], dw3 = h2^T go.
//
// The bf16 operands h1 and h2 are decided in FP64 where the FP32 activation
// lies next to a rounding boundary (about one in 3,900): the few that FP32
// decides the other way were most of the gradient's error against FP64 (6e-7
// to 1.6e-6 of its norm for 16,384 samples, as with one sample per thread).
//
// What bounds it: the activations (GELU and its slope, 64 per sample) on the
// vector ALUs, some 1,700 instructions per tile against 23 matrix products of
// 32 cycles.  16,384 samples: 64 workgroups of eight wavefronts, one tile each.
// One sample per thread on the vector ALUs with the sums read back from LDS
// took 86 us for that minibatch.
__global__ __launch_bounds__(kGradWG) void mlp_grad_kernel(const float *__restrict__ P, const float *__restrict__ raw,
                                                           const float *__restrict__ target, int64_t n,
                                                           float inv_scale, float *__restrict__ partial)
{
    constexpr size_t kTileBytes = sizeof(__bf16) * kGradWaves * kRows * kRow;
    constexpr size_t kRedBytes = sizeof(float) * kGradWaves * (kNParam + 1);
    __shared__ __align__(16) unsigned char smem[kTileBytes > kRedBytes ? kTileBytes : kRedBytes];
    __shared__ float sw[kNParam];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int m = lane & 31, h = lane >> 5;
    for (int k = threadIdx.x; k < kNParam; k += kGradWG) sw[k] = P[k];
    __syncthreads();
    // operands: W1 row m (both k halves), W2 row m and W2 column m in the
    // order in which the result registers hold the hidden units
    bf16x8_t w1, w2[2], w2t[2];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        w1[t] = t < kIn ? (__bf16)sw[kOffW1 + m * kIn + t] : (__bf16)0.f;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int unit = mlp_unit(8 * q + t, h);
            w2[q][t] = (__bf16)sw[kOffW2 + m * kH + unit];
            w2t[q][t] = (__bf16)sw[kOffW2 + unit * kH + m];
        }
    }
    bf16row_t *T = reinterpret_cast<bf16row_t *>(smem) + wv * kRows;
    f32x16_t dw2 = {}, dw1 = {}, db2 = {}, dw3 = {};
    float loss = 0.f, db3 = 0.f;
    const bf16x8_t zero = {};
    const int64_t ntile = (n + kTileS - 1) / kTileS;
    // every wavefront of the workgroup makes the same number of rounds
    for (int64_t t0 = (int64_t)blockIdx.x * kGradWaves; t0 < ntile; t0 += (int64_t)gridDim.x * kGradWaves) {
        const int64_t s = (t0 + wv) * kTileS + m;
        const bool act = s < n;
        // an opaque zero keeps the reads of biases and output weights inside
        // the loop: hoisted, they would hold ~60 registers
        int zo = 0;
        asm volatile("" : "+v"(zo));
        const float *sv = sw + 4 * h + zo;  // unit mlp_unit(j, h) is 8 (j / 4) + j % 4 further on
        // ---- forward
        bf16x8_t xb;
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const float r = act ? raw[s * kIn + k] : 0.f;
            xb[k] = (__bf16)((r - sw[kOffMean + k + zo]) * sw[kOffIstd + k + zo]);
        }
        xb[7] = (__bf16)0.f;
        if (h == 0) {
#pragma unroll
            for (int k = 0; k < kIn; ++k) T[kRowX + k][m] = xb[k];
            T[kRowX + kIn][m] = (__bf16)1.f;
        }
        f32x16_t z;
#pragma unroll
        for (int j = 0; j < 16; ++j) z[j] = sv[kOffB1 + mlp_unit(j, 0)];
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, h == 0 ? xb : zero, z, 0, 0, 0);
        float s1[16];  // slopes of layer 1
        bf16x8_t hb[2];
        uint32_t near = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            float g;
            gelu_and_slope(z[j], g, s1[j]);
            hb[j / 8][j % 8] = (__bf16)g;
            T[kRowH1 + mlp_unit(j, h)][m] = (__bf16)g;
            near |= act && near_boundary(g) ? 1u << j : 0u;
            // a few activations at a time: all sixteen in flight spill
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        if (__any(near != 0)) {
#pragma unroll 1
            while (near) {
                const int u = mlp_unit(__builtin_ctz(near), h);
                double zd = sw[kOffB1 + u];
#pragma unroll 1
                for (int k = 0; k < kIn; ++k)
                    zd = fma((double)bf16_round(sw[kOffW1 + u * kIn + k]), (double)(float)T[kRowX + k][m], zd);
                T[kRowH1 + u][m] = gelu_bf16(zd);
                near &= near - 1;
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) hb[j / 8][j % 8] = T[kRowH1 + mlp_unit(j, h)][m];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) z[j] = sv[kOffB2 + mlp_unit(j, 0)];
#pragma unroll
        for (int q = 0; q < 2; ++q) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2[q], hb[q], z, 0, 0, 0);
        float gz[16];  // w3 times the slope of layer 2
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            float g, sl;
            gelu_and_slope(z[j], g, sl);
            hb[j / 8][j % 8] = (__bf16)g;
            T[kRowH2 + mlp_unit(j, h)][m] = (__bf16)g;
            near |= act && near_boundary(g) ? 1u << j : 0u;
            gz[j] = bf16_round(sv[kOffW3 + mlp_unit(j, 0)]) * sl;
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (__any(near != 0)) {
#pragma unroll 1
            while (near) {
                const int u = mlp_unit(__builtin_ctz(near), h);
                double zd = sw[kOffB2 + u];
#pragma unroll 2
                for (int k = 0; k < kH; ++k)
                    zd = fma((double)bf16_round(sw[kOffW2 + u * kH + k]), (double)(float)T[kRowH1 + k][m], zd);
                T[kRowH2 + u][m] = gelu_bf16(zd);
                near &= near - 1;
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) hb[j / 8][j % 8] = T[kRowH2 + mlp_unit(j, h)][m];
        }
        float o = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) o = fmaf(bf16_round(sv[kOffW3 + mlp_unit(j, 0)]), (float)hb[j / 8][j % 8], o);
        o += __shfl_xor(o, 32, 64);  // the other half of the units
        o += sw[kOffB3];
        // ---- backward
        const float res = act ? (softplus_f(o) - target[s]) * inv_scale : 0.f;
        const float go = act ? 2.f * res * inv_scale * sigmoid_f(o) / (float)n : 0.f;
        if (h == 0) {
            loss += res * res;
            db3 += go;
            const Split3 g3 = split3(go);
#pragma unroll
            for (int p = 0; p < 3; ++p) T[kRowGo + p][m] = g3.p[p];
        }
        bf16x8_t gb[3][2];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const Split3 g3 = split3(go * gz[j]);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                gb[p][j / 8][j % 8] = g3.p[p];
                T[kRowG + 32 * p + mlp_unit(j, h)][m] = g3.p[p];
            }
        }
        f32x16_t ga = {};
#pragma unroll
        for (int p = 2; p >= 0; --p)
#pragma unroll
            for (int q = 0; q < 2; ++q) ga = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2t[q], gb[p][q], ga, 0, 0, 0);
        __syncthreads();
        // ---- sums over the tile's samples, 16 at a time
        bf16x8_t xc[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int s8 = 16 * c + 8 * h;
            const bf16x8_t h1 = row8(T[kRowH1 + m], s8);
            xc[c] = m < 8 ? row8(T[kRowX + (m & 7)], s8) : zero;
            const bf16x8_t gc = m < 3 ? row8(T[kRowGo + (m < 3 ? m : 0)], s8) : zero;
            dw3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row8(T[kRowH2 + m], s8), gc, dw3, 0, 0, 0);
#pragma unroll
            for (int p = 2; p >= 0; --p) {
                const bf16x8_t g = row8(T[kRowG + 32 * p + m], s8);
                dw2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g, h1, dw2, 0, 0, 0);
                db2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g, xc[c], db2, 0, 0, 0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const Split3 g3 = split3(ga[j] * s1[j]);
#pragma unroll
            for (int p = 0; p < 3; ++p) T[kRowG + 32 * p + mlp_unit(j, h)][m] = g3.p[p];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int p = 2; p >= 0; --p)
                dw1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row8(T[kRowG + 32 * p + m], 16 * c + 8 * h), xc[c], dw1, 0, 0,
                                                              0);
        __syncthreads();
    }
    // ---- the eight wavefronts' sums, in a fixed order
    float *red = reinterpret_cast<float *>(smem) + wv * (kNParam + 1);
    for (int k = lane; k < kOffW1; k += 64) red[k] = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {  // lane: column m of each product, rows = units
        const int u = mlp_unit(j, h);
        red[kOffW2 + u * kH + m] = dw2[j];
        if (m < kIn) red[kOffW1 + u * kIn + m] = dw1[j];
        if (m == kIn) {
            red[kOffB1 + u] = dw1[j];
            red[kOffB2 + u] = db2[j];
        }
        // the three parts of go sit in columns 0, 1, 2
        const float a = __shfl_down(dw3[j], 1, 64), b = __shfl_down(dw3[j], 2, 64);
        if (m == 0) red[kOffW3 + u] = (b + a) + dw3[j];
    }
    for (int d = 16; d > 0; d >>= 1) {
        loss += __shfl_xor(loss, d, 64);
        db3 += __shfl_xor(db3, d, 64);
    }
    if (lane == 0) {
        red[kOffB3] = db3;
        red[kNParam] = loss;
    }
    __syncthreads();
    const float *all = reinterpret_cast<const float *>(smem);
    for (int p = threadIdx.x; p <= kNParam; p += kGradWG) {
        float a = 0.f;
        for (int w = 0; w < kGradWaves; ++w) a += all[w * (kNParam + 1) + p];
        partial[(int64_t)blockIdx.x * (kNParam + 1) + p] = a;
    }
}

// grad[p] = sum over workgroups (fixed order: eight interleaved sums per
// parameter, then those in turn); loss = sum of squares / n.  32 parameters x
// 8 row groups per workgroup; one thread per parameter over all rows took 16
// us for 64 rows.
constexpr int kRedCols = 32, kRedRows = kWG / kRedCols;
__global__ __launch_bounds__(kWG) void mlp_grad_reduce_kernel(const float *__restrict__ partial, int nwg, int64_t n,
                                                               float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float s[kRedRows][kRedCols];
    const int c = threadIdx.x % kRedCols, g = threadIdx.x / kRedCols;
    const int p = blockIdx.x * kRedCols + c;
    float a = 0.f;
    if (p <= kNParam)
        for (int w = g; w < nwg; w += kRedRows) a += partial[(int64_t)w * (kNParam + 1) + p];
    s[g][c] = a;
    __syncthreads();
    if (g != 0 || p > kNParam) return;
    a = 0.f;
    for (int k = 0; k < kRedRows; ++k) a += s[k][c];
    if (p < kNParam)
        grad[p] = a;
    else
        *loss = a / (float)n;
}

__global__ __launch_bounds__(kWG) void mlp_adam_kernel(float *__restrict__ P, const float *__restrict__ g,
                                                        float *__restrict__ m, float *__restrict__ v, float lr,
                                                        float b1, float b2, float eps, float bc1, float bc2)
{
    const int p = blockIdx.x * kWG + threadIdx.x;
    if (p < kOffW1 || p >= kNParam) return;
    const float gi = g[p];
    const float mi = b1 * m[p] + (1.f - b1) * gi;
    const float vi = b2 * v[p] + (1.f - b2) * gi * gi;
    m[p] = mi;
    v[p] = vi;
    P[p] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// Standalone evaluation of the closure network with the same wavefront code
// (for parity tests): raw[n][7] -> out[n], flag[n] = 1 where the sweep would
// fall back to Smagorinsky.
__global__ __launch_bounds__(kWG) void mlp_forward_kernel(const MlpDev *net, const float *raw, int64_t n, float *out,
                                                          int32_t *flag)
{
    for (int64_t base = (int64_t)blockIdx.x * kWG; base < n; base += (int64_t)gridDim.x * kWG) {
        const int64_t s = base + threadIdx.x;
        const bool act = s < n;
        float x[7];
        bool bad = false;
        for (int k = 0; k < 7; ++k) {
            const float r = act ? raw[s * 7 + k] : 0.f;
            x[k] = (r - net->mean[k]) * net->istd[k];
            bad |= !(fabsf(x[k]) <= 8.f);
            if (!act) x[k] = 0.f;
        }
        const float o = mlp_forward_wave(net, x);
        if (act) {
            out[s] = o;
            flag[s] = (bad || !isfinite(o)) ? 1 : 0;
        }
    }
}

hipError_t launch_mlp_forward(const void *net, const float *raw, int64_t n, float *out, int32_t *flag, hipStream_t st)
{
    int64_t g = (n + kWG - 1) / kWG;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(mlp_forward_kernel, dim3((int)g), dim3(kWG), 0, st, reinterpret_cast<const MlpDev *>(net), raw,
                       n, out, flag);
    return hipGetLastError();
}

size_t mlp_grad_workspace_bytes(int64_t n)
{
    const int64_t nwg = (n + kWG - 1) / kWG;
    return (size_t)nwg * (kNParam + 1) * sizeof(float);
}

hipError_t launch_mlp_grad(const float *P, const float *raw, const float *target, int64_t n, float inv_scale,
                           float *grad, float *loss, float *work, hipStream_t st)
{
    // one workgroup per 256 samples (a row of the workspace each), up to two per CU
    const int64_t nwg = std::min<int64_t>((n + kGradWaves * kTileS - 1) / (kGradWaves * kTileS), kMaxGradWG);
    hipLaunchKernelGGL(mlp_grad_kernel, dim3((int)nwg), dim3(kGradWG), 0, st, P, raw, target, n, inv_scale, work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_grad_reduce_kernel, dim3((kNParam + 1 + kRedCols - 1) / kRedCols), dim3(kWG), 0, st, work,
                       (int)nwg, n, grad, loss);
    return hipGetLastError();
}

// Gradient pass without a caller workspace: the per-workgroup partials live in
// a library-owned device array of fixed size, one copy per GPU (each device
// gets its own instance of a __device__ variable).  Every workgroup writes its
// whole partial row before the reduction reads it, so nothing needs clearing
// between calls; calls that overlap on one GPU share the array and race.
constexpr int64_t kNoAllocMaxWG = kMlpNoAllocMaxSamples / kWG;
static_assert(kMlpNoAllocMaxSamples % kWG == 0, "whole workgroups");
static __device__ __align__(256) float scratch[kNoAllocMaxWG * (kNParam + 1)];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t mlp_scratch_address(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        // the array's name is a host-side stand-in: the device address of
        // this GPU's copy comes from the runtime, with this device current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_mlp_adam(float *P, const float *g, float *m, float *v, int64_t step, float lr, float b1, float b2,
                           float eps, hipStream_t st)
{
    const float bc1 = 1.f - powf(b1, (float)step), bc2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((kNParam + kWG - 1) / kWG), dim3(kWG), 0, st, P, g, m, v, lr, b1, b2, eps,
                       bc1, bc2);
    return hipGetLastError();
}

}  // namespace wlb

namespace wlb {

static uint16_t host_bf16_bits(float v)
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0x007fffffu) ? 0x40u : 0u));
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

size_t mlp_dev_bytes() { return sizeof(MlpDev); }

// Per-lane operand layout for mlp_forward_wave (see mlp.hpp): layer-1 A
// operand = W1 row (lane % 32) in both k halves; layer-2 A operand for
// k-chunk c = W2 row (lane % 32) at the hidden units that the B operand's
// k slots hold, unit(k = 8 h + t) = 16 c + 8 (t / 4) + 4 h + t % 4; layer-3 A
// operand = w3 at the same units, whatever the row.
void mlp_prepare(const float *P, void *out)
{
    MlpDev d;
    std::memset(&d, 0, sizeof d);
    for (int k = 0; k < kIn; ++k) {
        d.mean[k] = P[kOffMean + k];
        d.istd[k] = P[kOffIstd + k];
    }
    for (int lane = 0; lane < 64; ++lane) {
        const int m = lane % 32, h = lane / 32;
        for (int t = 0; t < 8; ++t) {
            d.w1[lane][t] = t < kIn ? host_bf16_bits(P[kOffW1 + m * kIn + t]) : 0;
            for (int c = 0; c < 2; ++c) {
                const int unit = 16 * c + 8 * (t / 4) + 4 * h + (t % 4);
                d.w2[c][lane][t] = host_bf16_bits(P[kOffW2 + m * kH + unit]);
                d.w3[c][h][t] = host_bf16_bits(P[kOffW3 + unit]);
            }
        }
    }
    for (int h = 0; h < 2; ++h)
        for (int j = 0; j < 16; ++j) {
            const int u = mlp_unit(j, h);
            d.b1[h][j] = P[kOffB1 + u];
            d.b2[h][j] = P[kOffB2 + u];
        }
    d.b3 = P[kOffB3];
    std::memcpy(out, &d, sizeof d);
}

}  // namespace wlb
