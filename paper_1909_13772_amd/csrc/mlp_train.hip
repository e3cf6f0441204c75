// mlp_train.hip -- training kernels of the learned closure network and the
// standalone forward evaluation.
//
// Loss over a minibatch of n samples: L = (1/n) sum_s ((softplus(o_s) - t_s)
// * inv_scale)^2, o = network output for the sample's raw features (see
// mlp.hpp for the network).  The forward/backward pass runs in FP32 with the
// GEMM operands (weights, x, h1, h2) rounded to bf16 exactly where the
// matrix-core forward rounds them, from FP32 values like there; the rounding
// has the straight-through gradient.  Every sum has one fixed order of FP32
// additions: over a layer's inputs in turn, over 64 samples in turn, over the
// four such sums of 256 samples, then over those (deterministic, and the same
// whatever the launch).  Adam keeps FP32 master weights; mean / inv_std are
// not trained.
#include <cstring>
#include <mutex>

#include "mlp.hpp"
#include "wlb_internal.hpp"

namespace wlb {

constexpr int kIn = 7, kH = 32;
constexpr int kOffMean = 0, kOffIstd = 7, kOffW1 = 14, kOffB1 = kOffW1 + kH * kIn, kOffW2 = kOffB1 + kH,
              kOffB2 = kOffW2 + kH * kH, kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH, kNParam = kOffB3 + 1;
static_assert(kNParam == 1359, "parameter count");
constexpr int kChunk = 64;       // samples of one chain of sums
constexpr int kGradWG = 1024;    // threads per kWG samples
static_assert(kWG == 4 * kChunk && kGradWG == 4 * kWG, "four chunks, four wavefronts for each");

// GELU and its slope at z, from one evaluation of the CDF's parts.
__device__ __forceinline__ void gelu_and_slope(float z, float &g, float &slope)
{
    const HalfErfc h = half_erfc_parts(z);
    g = fmaf(-(fabsf(z) * h.t), h.e, fmaxf(z, 0.f));
    const float tail = h.t * h.e;
    slope = (z >= 0.f ? 1.0f - tail : tail) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}
__device__ __forceinline__ float sigmoid_f(float o) { return 1.0f / (1.0f + expf(-o)); }

// One quantity of kWG samples for the kH units of a layer: rows of kH floats,
// whose quads are permuted by the sample so that one quad of 64 samples
// spreads over all banks.
struct alignas(16) UnitRows {
    float v[kWG][kH];
    __device__ __forceinline__ float4 &quad(int s, int k4) { return *reinterpret_cast<float4 *>(&v[s][((k4 ^ s) & 7) * 4]); }
    __device__ __forceinline__ float &at(int s, int k) { return v[s][(((k >> 2) ^ s) & 7) * 4 + (k & 3)]; }
};
// Shared memory of the gradient kernel.
struct alignas(16) GradLds {
    float w1[kH][8];             // bf16-rounded weights; the last column is not used
    float w2[kH][kH], w2t[kH][kH];
    float w3[kH], b1[kH], b2[kH];
    alignas(16) float go[kWG];   // d loss / d o
    alignas(16) float sq[kWG];   // squared residual
    alignas(16) float x[kWG][8]; // bf16-rounded features, then 1 (the inputs of W1 and b1)
    float b3;
    UnitRows h1, h2, gz1, gz2;   // activations and d loss / d z of both layers
};
static_assert(sizeof(GradLds) <= 160 * 1024 && sizeof(UnitRows) >= sizeof(float) * 4 * (kNParam + 1), "shared memory");

// Forward and backward pass of the network; one row of gradient partials per
// kWG samples, [gridDim.x][kNParam + 1] (last entry: sum of squared
// residuals).
//
// A layer's 256 x 32 outputs are shared out as two samples x four units per
// lane, all units of a wavefront the same: one broadcast read of four weights
// serves eight additions.  Forward products of two bf16 values are exact in
// FP32, so the fused multiply-add rounds like a product and a sum.  The
// parameter sums take one wavefront for rows 0..15 and one for rows 16..31 of
// W2 (4 x 2 sums per lane), one for W1 and b1 and one for the rest, per chunk;
// the wavefronts of a chunk run on one SIMD, so that the four SIMDs carry the
// same load.
//
// What bounds it: the vector ALUs of the CUs that have a workgroup (some 9,000
// instructions per 64 samples, two thirds of them the products and sums that
// are made one after the other).  With the reduction, us per call one after
// another: 16,384 samples 20.7, 262,144 samples 92; one thread per sample with
// all sums read back from LDS took 100 and 560 for the same bits.
__global__ __launch_bounds__(kGradWG) void mlp_grad_kernel(const float *__restrict__ P, const float *__restrict__ raw,
                                                           const float *__restrict__ target, int64_t n,
                                                           float inv_scale, float *__restrict__ partial)
{
    __shared__ __align__(16) GradLds L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t s0 = (int64_t)blockIdx.x * kWG;
    {
        const float w = bf16_round(P[kOffW2 + tid]);
        L.w2[tid / kH][tid % kH] = w;
        L.w2t[tid % kH][tid / kH] = w;
        if (tid < kH * kIn) L.w1[tid / kIn][tid % kIn] = bf16_round(P[kOffW1 + tid]);
        if (tid < kH) {
            L.w3[tid] = bf16_round(P[kOffW3 + tid]);
            L.b1[tid] = P[kOffB1 + tid];
            L.b2[tid] = P[kOffB2 + tid];
        }
        if (tid == 0) L.b3 = P[kOffB3];
        for (int e = tid; e < kWG * 8; e += kGradWG) {
            const int k = e & 7;
            const int64_t s = s0 + (e >> 3);
            float x = 1.f;
            if (k < kIn) x = bf16_round(((s < n ? raw[s * kIn + k] : 0.f) - P[kOffMean + k]) * P[kOffIstd + k]);
            L.x[e >> 3][k] = x;
        }
    }
    __syncthreads();
    // ---- forward
    const int u4 = wv & 7, u0 = 4 * u4;         // the lane's units
    const int sa = 128 * (wv >> 3) + lane;      // and samples sa, sa + 64
    float s1[2][4], s2[2][4];                   // slopes
    {
        float z[2][4] = {};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float4 xa = *reinterpret_cast<const float4 *>(&L.x[sa + 64 * r][0]);
            const float4 xb = *reinterpret_cast<const float4 *>(&L.x[sa + 64 * r][4]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float *w = L.w1[u0 + j];
                float a = fmaf(w[0], xa.x, 0.f);
                a = fmaf(w[1], xa.y, a);
                a = fmaf(w[2], xa.z, a);
                a = fmaf(w[3], xa.w, a);
                a = fmaf(w[4], xb.x, a);
                a = fmaf(w[5], xb.y, a);
                a = fmaf(w[6], xb.z, a);
                z[r][j] = a + L.b1[u0 + j];
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            float g[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) gelu_and_slope(z[r][j], g[j], s1[r][j]);
            L.h1.quad(sa + 64 * r, u4) = make_float4(bf16_round(g[0]), bf16_round(g[1]), bf16_round(g[2]), bf16_round(g[3]));
        }
    }
    __syncthreads();
    {
        float z[2][4] = {};
#pragma unroll 2
        for (int k4 = 0; k4 < kH / 4; ++k4) {
            const float4 h[2] = {L.h1.quad(sa, k4), L.h1.quad(sa + 64, k4)};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 w = *reinterpret_cast<const float4 *>(&L.w2[u0 + j][4 * k4]);
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    z[r][j] = fmaf(w.w, h[r].w, fmaf(w.z, h[r].z, fmaf(w.y, h[r].y, fmaf(w.x, h[r].x, z[r][j]))));
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            float g[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) gelu_and_slope(z[r][j] + L.b2[u0 + j], g[j], s2[r][j]);
            L.h2.quad(sa + 64 * r, u4) = make_float4(bf16_round(g[0]), bf16_round(g[1]), bf16_round(g[2]), bf16_round(g[3]));
        }
    }
    __syncthreads();
    if (tid < kWG) {
        const bool act = s0 + tid < n;
        float o = 0.f;
#pragma unroll
        for (int k4 = 0; k4 < kH / 4; ++k4) {
            const float4 h = L.h2.quad(tid, k4);
            const float4 w = *reinterpret_cast<const float4 *>(&L.w3[4 * k4]);
            o = fmaf(w.w, h.w, fmaf(w.z, h.z, fmaf(w.y, h.y, fmaf(w.x, h.x, o))));
        }
        o += L.b3;
        const float res = act ? (softplus_f(o) - target[s0 + tid]) * inv_scale : 0.f;
        L.go[tid] = act ? 2.f * res * inv_scale * sigmoid_f(o) / (float)n : 0.f;
        L.sq[tid] = res * res;
    }
    __syncthreads();
    // ---- backward
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float go = L.go[sa + 64 * r];
        float g[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) g[j] = go * L.w3[u0 + j] * s2[r][j];
        L.gz2.quad(sa + 64 * r, u4) = make_float4(g[0], g[1], g[2], g[3]);
    }
    __syncthreads();
    {
        float a[2][4] = {};
#pragma unroll 2
        for (int j4 = 0; j4 < kH / 4; ++j4) {
            const float4 g[2] = {L.gz2.quad(sa, j4), L.gz2.quad(sa + 64, j4)};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 w = *reinterpret_cast<const float4 *>(&L.w2t[u0 + k][4 * j4]);
#pragma unroll
                for (int r = 0; r < 2; ++r) a[r][k] = (((a[r][k] + g[r].x * w.x) + g[r].y * w.y) + g[r].z * w.z) + g[r].w * w.w;
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
            L.gz1.quad(sa + 64 * r, u4) =
                make_float4(a[r][0] * s1[r][0], a[r][1] * s1[r][1], a[r][2] * s1[r][2], a[r][3] * s1[r][3]);
    }
    __syncthreads();
    // ---- parameter sums over the chunk's samples, one after the other
    const int role = wv >> 2, chunk = wv & 3, q0 = chunk * kChunk;
    float a[4][2] = {};
    float loss = 0.f;
    const int r4 = role < 2 ? 4 * role + (lane >> 4) : lane >> 3;          // rows 4 r4 ... of W2, W1
    const int c0 = role < 2 ? 2 * (lane & 15) : role == 2 ? lane & 7 : lane & 31;  // first column
    // q0 is a multiple of 8: eight samples at a time, the places of a row's
    // quads are the same eight for every group
    if (role < 2) {
#pragma unroll 8
        for (int q = q0; q < q0 + kChunk; ++q) {
            const float4 g = L.gz2.quad(q, r4);
            const float2 h = *reinterpret_cast<const float2 *>(&L.h1.at(q, c0));
            a[0][0] += g.x * h.x;
            a[0][1] += g.x * h.y;
            a[1][0] += g.y * h.x;
            a[1][1] += g.y * h.y;
            a[2][0] += g.z * h.x;
            a[2][1] += g.z * h.y;
            a[3][0] += g.w * h.x;
            a[3][1] += g.w * h.y;
        }
    } else if (role == 2) {
#pragma unroll 8
        for (int q = q0; q < q0 + kChunk; ++q) {
            const float4 g = L.gz1.quad(q, r4);
            const float x = L.x[q][c0];
            a[0][0] += g.x * x;
            a[1][0] += g.y * x;
            a[2][0] += g.z * x;
            a[3][0] += g.w * x;
        }
    } else {
        // lanes 0..31: b2; lanes 32..63: w3; every lane: b3
        UnitRows &V = lane < kH ? L.gz2 : L.h2;
#pragma unroll 8
        for (int q = q0; q < q0 + kChunk; ++q) {
            const float go = L.go[q];
            a[0][0] += V.at(q, c0) * (lane < kH ? 1.f : go);
            a[1][0] += go;
        }
        if (chunk == 0)
#pragma unroll 8
            for (int q = 0; q < kWG; q += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(&L.sq[q]);
                loss = (((loss + v.x) + v.y) + v.z) + v.w;
            }
    }
    __syncthreads();
    // ---- the four chunks' sums in turn
    float(*red)[kNParam + 1] = reinterpret_cast<float(*)[kNParam + 1]>(&L.gz1);
    float *out = red[chunk];
    if (role < 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            out[kOffW2 + (4 * r4 + j) * kH + c0] = a[j][0];
            out[kOffW2 + (4 * r4 + j) * kH + c0 + 1] = a[j][1];
        }
    } else if (role == 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[c0 < kIn ? kOffW1 + (4 * r4 + j) * kIn + c0 : kOffB1 + 4 * r4 + j] = a[j][0];
    } else {
        out[(lane < kH ? kOffB2 : kOffW3) + c0] = a[0][0];
        if (lane == 0) {
            out[kOffB3] = a[1][0];
            if (chunk == 0) L.sq[0] = loss;
        }
    }
    __syncthreads();
    float *row = partial + (int64_t)blockIdx.x * (kNParam + 1);
    for (int p = tid; p <= kNParam; p += kGradWG) {
        float r = 0.f;
        if (p == kNParam)
            r = L.sq[0];
        else if (p >= kOffW1)
            for (int c = 0; c < 4; ++c) r += red[c][p];
        row[p] = r;
    }
}

// grad[p] = sum over workgroups in turn; loss = sum of squares / n.  A
// workgroup takes 32 parameters and brings 256 rows of theirs into LDS at a
// time, from where one thread each adds them up: the additions wait for one
// another, the loads do not.
constexpr int kRedCols = 32, kRedRows = 256;
__global__ __launch_bounds__(kWG) void mlp_grad_reduce_kernel(const float *__restrict__ partial, int64_t nwg, int64_t n,
                                                               float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float s[kRedRows][kRedCols];
    const int c = threadIdx.x % kRedCols, g = threadIdx.x / kRedCols;
    const int p = blockIdx.x * kRedCols + c;
    float a = 0.f;
    for (int64_t w0 = 0; w0 < nwg; w0 += kRedRows) {
        const int rows = nwg - w0 < kRedRows ? (int)(nwg - w0) : kRedRows;
        if (p <= kNParam)
#pragma unroll 8
            for (int w = g; w < rows; w += kWG / kRedCols) s[w][c] = partial[(w0 + w) * (kNParam + 1) + p];
        __syncthreads();
        if (g == 0 && p <= kNParam)
#pragma unroll 16
            for (int w = 0; w < rows; ++w) a += s[w][c];
        __syncthreads();
    }
    if (g != 0 || p > kNParam) return;
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
    const int64_t nwg = (n + kWG - 1) / kWG;
    hipLaunchKernelGGL(mlp_grad_kernel, dim3((int)nwg), dim3(kGradWG), 0, st, P, raw, target, n, inv_scale, work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_grad_reduce_kernel, dim3((kNParam + 1 + kRedCols - 1) / kRedCols), dim3(kWG), 0, st, work,
                       nwg, n, grad, loss);
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
