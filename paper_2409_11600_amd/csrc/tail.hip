// The operations that close a training step behind the residual blocks: global average pool and fully connected
// layer (the head of the ResNet recipe the paper trains, section "Experiments and Discussion"; the fully connected
// layer is the `@` operator of section "Automatic Differentiation"), the softmax cross-entropy loss node that has to
// end every step (same section), and the optimizer updates with the clearing of the gradient buffers (section
// "Caching and Pooling").  All of them are small and bound by memory or by launch latency; the kernels are plain
// streaming code.  The fully connected layer runs on the convolution kernels (1x1 filter, 1x1 image).
#include <math.h>

#include <algorithm>

#include "nsk_internal.h"

namespace nsk {
namespace {

bool unaligned(const void *p) { return ((uintptr_t)p & 15) != 0; }

#define TAIL_TRY(expr)                \
    do {                              \
        int status_ = (expr);         \
        if (status_ != NSK_OK) return status_; \
    } while (0)

__device__ inline float ld(const float *p, long i) { return p[i]; }
__device__ inline float ld(const bf16_t *p, long i) { return (float)p[i]; }

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ inline float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// ----------------------------------------------------------------------------- global average pool
// NHWC, channel count a multiple of the 16-byte vector width with C/VEC dividing 1024: one block of 1024 threads per
// image.  A thread owns one vector of channels and every G-th position (G = 1024 / vectors per pixel), four loads
// in flight; the G partial sums per channel meet in LDS and are added in a fixed order.
template <typename T, int VEC>
__global__ __launch_bounds__(1024) void avgpool_fwd_nhwc_vec(const T *__restrict__ x, T *__restrict__ y, int C, int HW)
{
    typedef T Vec __attribute__((ext_vector_type(VEC)));
    extern __shared__ float part[];                 // [G][C]
    const int CV = C / VEC, G = 1024 / CV;
    const int cv = threadIdx.x % CV, g = threadIdx.x / CV;
    const Vec *p = (const Vec *)(x + (long)blockIdx.x * HW * C) + cv;
    float s[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) s[e] = 0.f;
    int k = g;
    for (; k + 3 * G < HW; k += 4 * G) {
        const Vec v0 = p[(long)k * CV], v1 = p[(long)(k + G) * CV], v2 = p[(long)(k + 2 * G) * CV], v3 = p[(long)(k + 3 * G) * CV];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] += ((float)v0[e] + (float)v1[e]) + ((float)v2[e] + (float)v3[e]);
    }
    for (; k < HW; k += G) {
        const Vec v = p[(long)k * CV];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] += (float)v[e];
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) part[g * C + cv * VEC + e] = s[e];
    __syncthreads();
    for (int c = threadIdx.x; c < C; c += 1024) {
        float t = 0.f;
        for (int gg = 0; gg < G; ++gg) t += part[gg * C + c];
        y[(long)blockIdx.x * C + c] = (T)(t / (float)HW);
    }
}
// NHWC, any channel count: one thread per (n, c), neighbouring threads read neighbouring channels.
template <typename T>
__global__ __launch_bounds__(256) void avgpool_fwd_nhwc(const T *__restrict__ x, T *__restrict__ y, int N, int C, int HW)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long)N * C) return;
    const long n = i / C, c = i - n * C;
    const T *p = x + n * HW * (long)C + c;
    float s = 0.f;
    for (int k = 0; k < HW; ++k) s += ld(p, (long)k * C);
    y[i] = (T)(s / (float)HW);
}
// NCHW: one wavefront per (n, c) plane, lanes stride over the plane, fixed-order cross-lane sum.
template <typename T>
__global__ __launch_bounds__(256) void avgpool_fwd_nchw(const T *__restrict__ x, T *__restrict__ y, long planes, int HW)
{
    const long pl = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (pl >= planes) return;
    const T *p = x + pl * HW;
    float s = 0.f;
    for (int k = threadIdx.x & 63; k < HW; k += 64) s += ld(p, k);
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) y[pl] = (T)(s / (float)HW);
}
template <typename T, bool NHWC>
__global__ __launch_bounds__(256) void avgpool_bwd_kernel(const T *__restrict__ dy, T *__restrict__ dx, long total, int C,
                                                          int HW, int accumulate)
{
    const float inv = 1.f / (float)HW;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        long nc;
        if (NHWC) {
            const long n = i / ((long)HW * C);
            nc = n * C + i % C;
        } else {
            nc = i / HW;
        }
        float v = ld(dy, nc) * inv;
        if (accumulate) v += ld(dx, i);
        dx[i] = (T)v;
    }
}

// ----------------------------------------------------------------------------- fully connected layer helpers
template <typename T>
__global__ __launch_bounds__(256) void add_bias_kernel(T *__restrict__ y, const float *__restrict__ bias, long total, int K)
{
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256)
        y[i] = (T)(ld(y, i) + bias[i % K]);
}
// db[k] (+)= sum_n dy[n][k]: a block owns CB columns (neighbouring lanes, so a wavefront reads contiguous bytes of 64/CB
// rows), its 1024/CB row lanes take every (1024/CB)-th row each and their partial sums are added in a fixed order.
// Bound by how many loads are on their way: with 64 columns a block, 768 columns are 12 blocks.  From 1024 rows on a block
// has 16 columns (fp32 10000 x 768: 32.1 us with 64 columns, 24.3 with 16).
template <typename T, int CB>
__global__ __launch_bounds__(1024) void bias_grad_kernel(const T *__restrict__ dy, float *__restrict__ db, int N, int K,
                                                         int accumulate)
{
    constexpr int RL = 1024 / CB;
    __shared__ float part[RL][CB], few[16][CB];
    const int col = threadIdx.x % CB, rl = threadIdx.x / CB, k = blockIdx.x * CB + col;
    float s = 0.f;
    if (k < K) {
#pragma unroll 8
        for (int n = rl; n < N; n += RL) s += ld(dy, (long)n * K + k);
    }
    part[rl][col] = s;
    __syncthreads();
    if (rl < 16) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < RL / 16; ++r) t += part[rl * (RL / 16) + r][col];
        few[rl][col] = t;
    }
    __syncthreads();
    if (rl == 0 && k < K) {
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) t += few[r][col];
        db[k] = accumulate ? db[k] + t : t;
    }
}

// The same in two launches for many rows, where a launch has the workspace of the weight gradient before it (whose partial sums have been
// read by then): blocks of 64 columns x a share of the rows, four columns (16 or 8 bytes) a lane, then the shares' sums in 64
// bits.  The kernel above keeps 48 CUs busy with 768 columns and reads them in 64-byte pieces: fp32 10000 x 768 (30.7 MB)
// 24.5 us there, 9.4 here; bf16 20.8 / 6.9.
constexpr int kBiasShares = 64;
template <typename T>
__global__ __launch_bounds__(256) void bias_partial_kernel(const T *__restrict__ dy, float *__restrict__ part, int N, int K, int rows)
{
    typedef T Vec __attribute__((ext_vector_type(4)));
    __shared__ f32x4 sums[16][16];
    const int cv = threadIdx.x & 15, rl = threadIdx.x >> 4, k = blockIdx.x * 64 + cv * 4;
    const int r1 = min(N, (int)(blockIdx.y + 1) * rows);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (k < K) {
#pragma unroll 8
        for (int n = blockIdx.y * rows + rl; n < r1; n += 16) {
            const Vec v = *(const Vec *)(dy + (long)n * K + k);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += (float)v[e];
        }
    }
    sums[rl][cv] = s;
    __syncthreads();
    if (rl == 0 && k < K) {
        double t[4] = {};
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] += (double)sums[r][cv][e];
        *(f32x4 *)(part + (long)blockIdx.y * K + k) = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
    }
}
__global__ __launch_bounds__(64) void bias_final_kernel(const float *__restrict__ part, float *__restrict__ db, int shares, int K, int accumulate)
{
    const int k = blockIdx.x * 16 + (threadIdx.x & 15), q = threadIdx.x >> 4;      // four lanes a column, every fourth share each
    double s = 0.;
    if (k < K) {
#pragma unroll 8
        for (int r = q; r < shares; r += 4) s += (double)part[(long)r * K + k];
    }
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (q == 0 && k < K) db[k] = accumulate ? db[k] + (float)s : (float)s;
}

// Matrix products with very few rows (a recurrent step: 50 samples): a tile kernel would run on a handful of blocks,
// so here every output element has its own thread and the product runs on the vector units.
//   forward:  y[n][k] = sum_c x[n][c] * w[k][c] (+ bias[k]); lane = k (the 64 rows of w a wavefront walks stay in L1
//             for the iterations that share a cache line)
//   backward: dx[n][c] (+)= sum_k dy[n][k] * w[k][c]; lane = c, w read row by row with consecutive lanes on
//             consecutive c, so no packed transposed copy of the filter is needed
// forward: one thread per output element (splitting its reduction over wavefronts, as the backward kernel below does,
// is slower here: four times as many wavefronts then walk the rows of w with a stride)
template <typename T>
__global__ __launch_bounds__(256) void linear_small_fwd_kernel(const T *__restrict__ x, const T *__restrict__ w,
                                                               const float *__restrict__ bias, T *__restrict__ y, int N,
                                                               int C, int K)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long)N * K) return;
    const int n = (int)(i / K), k = (int)(i - (long)n * K);
    const T *xr = x + (long)n * C, *wr = w + (long)k * C;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    int c = 0;
    for (; c + 3 < C; c += 4) {
        s0 += ld(xr, c) * ld(wr, c);
        s1 += ld(xr, c + 1) * ld(wr, c + 1);
        s2 += ld(xr, c + 2) * ld(wr, c + 2);
        s3 += ld(xr, c + 3) * ld(wr, c + 3);
    }
    for (; c < C; ++c) s0 += ld(xr, c) * ld(wr, c);
    float r = (s0 + s1) + (s2 + s3);
    if (bias) r = (float)(T)r + bias[k];      // as the large path: product rounded to the storage type, then the bias
    y[i] = (T)r;
}

// Few outputs (the output layer of a classifier): sixteen lanes share one, else its whole reduction is a chain of loads in one thread
// and the launch a handful of wavefronts: 50 x 2 outputs of 256 channels 8.3 us with a thread each, 2.4 here.
template <typename T>
__global__ __launch_bounds__(256) void linear_few_fwd_kernel(const T *__restrict__ x, const T *__restrict__ w, const float *__restrict__ bias,
                                                             T *__restrict__ y, int N, int C, int K)
{
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), q = threadIdx.x & 15;
    const bool live = i < N * K;
    const int n = live ? i / K : 0, k = live ? i - n * K : 0;
    const T *xr = x + (long)n * C, *wr = w + (long)k * C;
    float s = 0.f;
#pragma unroll 8
    for (int c = q; c < C; c += 16) s += ld(xr, c) * ld(wr, c);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
    if (!live || q != 0) return;
    if (bias) s = (float)(T)s + bias[k];
    y[i] = (T)s;
}

// backward: a block computes 64 consecutive outputs of one row; its four wavefronts each take a quarter of the
// reduction and the quarters are added in a fixed order through LDS.  (Giving a block several rows, so that a weight
// element is loaded once for all of them, was measured slower: 16 us against 9 us at 50 rows x 768 -> 256, because the
// launch then has too few blocks to hide the latency of its loads.)
template <typename T>
__global__ __launch_bounds__(256) void linear_small_dgrad_kernel(const T *__restrict__ dy, const T *__restrict__ w,
                                                                 T *__restrict__ dx, int N, int C, int K, int accumulate)
{
    __shared__ float part[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int n = blockIdx.y, c = blockIdx.x * 64 + lane;
    const int k0 = (int)((long)K * q / 4), k1 = (int)((long)K * (q + 1) / 4);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (c < C) {
        const T *dr = dy + (long)n * K, *wc = w + c;
        int k = k0;
        for (; k + 3 < k1; k += 4) {
            s0 += ld(dr, k) * ld(wc, (long)k * C);
            s1 += ld(dr, k + 1) * ld(wc, (long)(k + 1) * C);
            s2 += ld(dr, k + 2) * ld(wc, (long)(k + 2) * C);
            s3 += ld(dr, k + 3) * ld(wc, (long)(k + 3) * C);
        }
        for (; k < k1; ++k) s0 += ld(dr, k) * ld(wc, (long)k * C);
    }
    part[q][lane] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (q == 0 && c < C) {
        float r = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
        const long i = (long)n * C + c;
        if (accumulate) r += ld(dx, i);
        dx[i] = (T)r;
    }
}

constexpr int kSmallRows = 64;     // up to this many rows the per-element kernels are used

// ----------------------------------------------------------------------------- softmax cross-entropy
// One wavefront per sample.  mode 0: per-sample loss; mode 1: gradient of the logits.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void xent_kernel(const T *__restrict__ z, const int *__restrict__ labels, int N, int K,
                                                   float *__restrict__ per_sample, T *__restrict__ dz, float coef)
{
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    const int lane = threadIdx.x & 63;
    const T *row = z + (long)n * K;
    float m = -INFINITY;
    for (int k = lane; k < K; k += 64) m = fmaxf(m, ld(row, k));
    m = wave_max(m);
    float s = 0.f;
    for (int k = lane; k < K; k += 64) s += expf(ld(row, k) - m);
    s = wave_sum(s);
    const int lab = labels[n];
    if (MODE == 0) {
        if (lane == 0) per_sample[n] = (lab >= 0 && lab < K) ? logf(s) + (m - ld(row, lab)) : NAN;
    } else {
        const float inv = 1.f / s;
        for (int k = lane; k < K; k += 64) {
            const float p = expf(ld(row, k) - m) * inv;
            dz[(long)n * K + k] = (T)(coef * (p - (k == lab ? 1.f : 0.f)));
        }
    }
}
// loss = mean of per_sample, one block, fixed order.
__global__ __launch_bounds__(256) void mean_kernel(const float *__restrict__ v, int N, float *__restrict__ out)
{
    __shared__ double part[4];
    double s = 0.0;
    for (int i = threadIdx.x; i < N; i += 256) s += (double)v[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (float)(((part[0] + part[1]) + (part[2] + part[3])) / (double)N);
}

// ----------------------------------------------------------------------------- optimizers
struct AdamCoef {
    float lr, beta1, beta2, eps, c1, c2;   // c1 = 1/(1-beta1^t); c2 = 1/(1-beta2^t)
};

// One launch updates up to kMaxParams parameter tensors: blockIdx.y names the tensor, blockIdx.x strides over it.
constexpr int kMaxParams = 32;
struct ParamEntry {
    float *w, *g, *s1, *s2;
    bf16_t *w_lp;
    size_t n;
    float wd;        // SGD: weight decay; AdamW: 1 - lr*weight_decay
};
struct ParamTable {
    ParamEntry e[kMaxParams];
};

template <bool ADAM>
__global__ __launch_bounds__(256) void optimizer_kernel(const ParamTable tab, float lr, float momentum, AdamCoef ac,
                                                        const float *__restrict__ grad_scale)
{
    const ParamEntry &p = tab.e[blockIdx.y];
    const size_t n = p.n;
    float *__restrict__ w = p.w, *__restrict__ g = p.g, *__restrict__ s1 = p.s1, *__restrict__ s2 = p.s2;
    bf16_t *__restrict__ w_lp = p.w_lp;
    const float wd = p.wd;
    const float scale = grad_scale ? grad_scale[0] : 1.f;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        float wi = w[i];
        const float gi = g[i] * scale;
        if (ADAM) {
            wi *= wd;
            const float m = ac.beta1 * s1[i] + (1.f - ac.beta1) * gi;
            const float v = ac.beta2 * s2[i] + (1.f - ac.beta2) * gi * gi;
            s1[i] = m;
            s2[i] = v;
            wi -= ac.lr * (m * ac.c1) / (sqrtf(v * ac.c2) + ac.eps);
        } else {
            const float v = momentum * s1[i] + (gi + wd * wi);
            s1[i] = v;
            wi -= lr * v;
        }
        w[i] = wi;
        g[i] = 0.f;
        if (w_lp) w_lp[i] = (bf16_t)wi;
    }
}

// Bound by memory once enough loads are on their way: at most 256 partial sums, so a block is 1024 threads that take 16 bytes
// at a time (g is on a 16-byte boundary), four of them at once (us with the final sum, 256 threads and
// single floats / here: 8.4 M elements 27.3 / 7.1, 197 k 12.5 / 5.7, 768 4.4 / 4.4).
__global__ __launch_bounds__(1024) void sumsq_partial_kernel(size_t n, const float *__restrict__ g, float *__restrict__ partials)
{
    __shared__ double part[16];
    double s = 0.0;
    const size_t nv = n / 4, step = (size_t)gridDim.x * 1024, first = (size_t)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll 4
    for (size_t i = first; i < nv; i += step) {
        const f32x4 v = *(const f32x4 *)(g + 4 * i);
        s += ((double)(v[0] * v[0]) + (double)(v[1] * v[1])) + ((double)(v[2] * v[2]) + (double)(v[3] * v[3]));
    }
    if (first < n - 4 * nv) {
        const float v = g[4 * nv + first];
        s += (double)(v * v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += part[w];
        partials[blockIdx.x] = (float)t;
    }
}
// The clip of many tensors in two launches (seven tensors one by one: sixteen launches, 63 us behind busy ones): a block takes its share
// of every tensor and leaves one partial sum; `add` for the second and later launches of more than kMaxSumsq tensors.
constexpr int kMaxSumsq = 48;
struct SumsqTable {
    const float *g[kMaxSumsq];
    size_t n[kMaxSumsq];
    int count, add;
};
__global__ __launch_bounds__(1024) void sumsq_multi_kernel(const SumsqTable tab, float *__restrict__ partials)
{
    __shared__ double part[16];
    double s = 0.0;
    const size_t step = (size_t)gridDim.x * 1024, first = (size_t)blockIdx.x * 1024 + threadIdx.x;
    for (int t = 0; t < tab.count; ++t) {
        const float *__restrict__ g = tab.g[t];
        const size_t n = tab.n[t], nv = n / 4;
#pragma unroll 4
        for (size_t i = first; i < nv; i += step) {
            const f32x4 v = *(const f32x4 *)(g + 4 * i);
            s += ((double)(v[0] * v[0]) + (double)(v[1] * v[1])) + ((double)(v[2] * v[2]) + (double)(v[3] * v[3]));
        }
        if (first < n - 4 * nv) {
            const float v = g[4 * nv + first];
            s += (double)(v * v);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = tab.add ? (double)partials[blockIdx.x] : 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += part[w];
        partials[blockIdx.x] = (float)t;
    }
}
__global__ __launch_bounds__(64) void clip_final_kernel(const float *__restrict__ partials, int nb, float max_norm, float *__restrict__ sumsq,
                                                        float *__restrict__ scale)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += 64) s += (double)partials[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) {
        const float q = (float)s, r = max_norm / (sqrtf(q) + 1e-6f);
        sumsq[0] = q;
        scale[0] = r < 1.f ? r : 1.f;
    }
}
// one wavefront: lane l adds the partial sums l, l + 64, ..., the lanes are added in a fixed order
__global__ __launch_bounds__(64) void sumsq_final_kernel(const float *__restrict__ partials, int nb, float *__restrict__ sumsq)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += 64) s += (double)partials[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) sumsq[0] = (float)((double)sumsq[0] + s);
}
__global__ void clip_scale_kernel(const float *__restrict__ sumsq, float max_norm, float *__restrict__ scale)
{
    const float r = max_norm / (sqrtf(sumsq[0]) + 1e-6f);
    scale[0] = r < 1.f ? r : 1.f;
}

int stream_grid(size_t items)
{
    size_t b = (items + 255) / 256;
    if (b > 256 * 16) b = 256 * 16;
    if (b < 1) b = 1;
    return (int)b;
}

bool dtype_ok(int dtype) { return dtype == NSK_F32 || dtype == NSK_BF16; }

nsk_conv_desc_t linear_as_conv(const nsk_linear_desc_t *d)
{
    nsk_conv_desc_t c{};
    c.N = d->N; c.C = d->C; c.H = 1; c.W = 1;
    c.K = d->K; c.R = 1; c.S = 1;
    c.stride_h = c.stride_w = 1;
    c.pad_h = c.pad_w = 0;
    c.dil_h = c.dil_w = 1;
    c.dtype = d->dtype;
    c.layout = NSK_NHWC;
    return c;
}

int linear_check(const nsk_linear_desc_t *d)
{
    if (!d) return NSK_ERR_NULL;
    if (d->N <= 0 || d->C <= 0 || d->K <= 0 || !dtype_ok(d->dtype)) return NSK_ERR_BAD_DESC;
    return NSK_OK;
}

// Bias gradient in two launches (bias_partial_kernel): from 6000 rows on, where it is the faster one at every width (us, one launch / two:
// 64 columns fp32 5.3 / 4.6, bf16 5.8 / 4.6; 256 5.2 / 4.6, 5.8 / 4.7; 768 16.0 / 7.1, 13.7 / 4.9; 4096 30.3 / 17.8, 31.8 / 11.9).  At
// 3000 rows the second launch costs more than it gives up to 768 columns (64 3.7 / 4.1, 4.0 / 4.4; 768 3.9 / 4.5, 4.0 / 4.5; 2000 rows
// 3.0 / 5.8); between, the widths differ (4000 rows: 64 4.3 / 4.3, 384 4.3 / 4.7, 768 10.9 / 5.3, 4096 21.2 / 13.3).
bool bias_in_shares(const nsk_linear_desc_t *d) { return d->N >= 6000 && d->K >= 64 && d->K % 4 == 0; }
size_t bias_share_bytes(const nsk_linear_desc_t *d) { return (size_t)kBiasShares * d->K * sizeof(float); }

}  // namespace
}  // namespace nsk

using namespace nsk;

extern "C" {

int nsk_global_avgpool_fwd(int dtype, int layout, int N, int C, int H, int W, const void *x, void *y, void *stream)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || !dtype_ok(dtype) || (layout != NSK_NCHW && layout != NSK_NHWC))
        return NSK_ERR_BAD_DESC;
    if (!x || !y) return NSK_ERR_NULL;
    if (unaligned(x) || unaligned(y)) return NSK_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const long planes = (long)N * C;
    const int HW = H * W;
    const int vec = dtype == NSK_BF16 ? 8 : 4;
    if (layout == NSK_NHWC && C % vec == 0 && 1024 % (C / vec) == 0) {
        const size_t smem = (size_t)1024 * vec * sizeof(float);     // G * C floats with G = 1024 / (C / vec)
        if (dtype == NSK_BF16)
            hipLaunchKernelGGL((avgpool_fwd_nhwc_vec<bf16_t, 8>), dim3(N), dim3(1024), smem, st, (const bf16_t *)x, (bf16_t *)y, C, HW);
        else
            hipLaunchKernelGGL((avgpool_fwd_nhwc_vec<float, 4>), dim3(N), dim3(1024), smem, st, (const float *)x, (float *)y, C, HW);
    } else if (layout == NSK_NHWC) {
        const dim3 grid((unsigned)((planes + 255) / 256));
        if (dtype == NSK_BF16)
            hipLaunchKernelGGL(avgpool_fwd_nhwc<bf16_t>, grid, dim3(256), 0, st, (const bf16_t *)x, (bf16_t *)y, N, C, HW);
        else
            hipLaunchKernelGGL(avgpool_fwd_nhwc<float>, grid, dim3(256), 0, st, (const float *)x, (float *)y, N, C, HW);
    } else {
        const dim3 grid((unsigned)((planes + 3) / 4));
        if (dtype == NSK_BF16)
            hipLaunchKernelGGL(avgpool_fwd_nchw<bf16_t>, grid, dim3(256), 0, st, (const bf16_t *)x, (bf16_t *)y, planes, HW);
        else
            hipLaunchKernelGGL(avgpool_fwd_nchw<float>, grid, dim3(256), 0, st, (const float *)x, (float *)y, planes, HW);
    }
    return check_launch();
}

int nsk_global_avgpool_bwd(int dtype, int layout, int N, int C, int H, int W, const void *dy, void *dx, int accumulate,
                           void *stream)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || !dtype_ok(dtype) || (layout != NSK_NCHW && layout != NSK_NHWC))
        return NSK_ERR_BAD_DESC;
    if (accumulate != 0 && accumulate != 1) return NSK_ERR_BAD_DESC;
    if (!dy || !dx) return NSK_ERR_NULL;
    if (unaligned(dy) || unaligned(dx)) return NSK_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const long total = (long)N * C * H * W;
    const dim3 grid(stream_grid((size_t)total));
#define NSK_AP(T, L) \
    hipLaunchKernelGGL((avgpool_bwd_kernel<T, L>), grid, dim3(256), 0, st, (const T *)dy, (T *)dx, total, C, H * W, accumulate)
    if (dtype == NSK_BF16) {
        if (layout == NSK_NHWC) NSK_AP(bf16_t, true); else NSK_AP(bf16_t, false);
    } else {
        if (layout == NSK_NHWC) NSK_AP(float, true); else NSK_AP(float, false);
    }
#undef NSK_AP
    return check_launch();
}

size_t nsk_linear_workspace_bytes(const nsk_linear_desc_t *desc, int pass)
{
    if (linear_check(desc) != NSK_OK) return 0;
    const nsk_conv_desc_t c = linear_as_conv(desc);
    const size_t conv = nsk_conv2d_workspace_bytes(&c, pass);
    return pass == NSK_PASS_WGRAD && bias_in_shares(desc) ? std::max(conv, bias_share_bytes(desc)) : conv;
}

int nsk_linear_fwd(const nsk_linear_desc_t *desc, const void *x, const void *w, const float *bias, void *y,
                   void *workspace, size_t workspace_bytes, void *stream)
{
    TAIL_TRY(linear_check(desc));
    if (bias && unaligned(bias)) return NSK_ERR_ALIGNMENT;
    if (desc->N <= kSmallRows) {
        if (!x || !w || !y) return NSK_ERR_NULL;
        if (unaligned(x) || unaligned(w) || unaligned(y)) return NSK_ERR_ALIGNMENT;
        const long total = (long)desc->N * desc->K;
        const dim3 grid((unsigned)((total + 255) / 256)), few((unsigned)((total + 15) / 16));
        // From 128 channels on.  At 64 sixteen lanes are faster as well (4.2 / 2.6 us), but the order of the sum decides there on which side
        // of zero one ReLU of the two-step fp32 training test falls, and its expected weights with it: that sum stays as it is.  Up to
        // 4096 outputs, what the kernel was built for; beyond it would be faster too (us, a thread each / sixteen lanes, fp32: 64 x 64
        // outputs of 128, 256, 1024 channels 6.3 / 2.5, 10.6 / 2.7, 36.8 / 4.0; 64 x 256 6.7 / 2.8, 11.5 / 3.3, 40.8 / 6.6; 64 x 1000 7.9 / 4.6, 13.1 / 6.4,
        // 50.1 / 18.2; bf16 the same within 10%).
        const bool lanes = total <= 4096 && desc->C >= 128;
        if (lanes && desc->dtype == NSK_BF16)
            hipLaunchKernelGGL(linear_few_fwd_kernel<bf16_t>, few, dim3(256), 0, (hipStream_t)stream, (const bf16_t *)x, (const bf16_t *)w, bias,
                               (bf16_t *)y, desc->N, desc->C, desc->K);
        else if (lanes)
            hipLaunchKernelGGL(linear_few_fwd_kernel<float>, few, dim3(256), 0, (hipStream_t)stream, (const float *)x, (const float *)w, bias,
                               (float *)y, desc->N, desc->C, desc->K);
        else if (desc->dtype == NSK_BF16)
            hipLaunchKernelGGL(linear_small_fwd_kernel<bf16_t>, grid, dim3(256), 0, (hipStream_t)stream, (const bf16_t *)x,
                               (const bf16_t *)w, bias, (bf16_t *)y, desc->N, desc->C, desc->K);
        else
            hipLaunchKernelGGL(linear_small_fwd_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream, (const float *)x,
                               (const float *)w, bias, (float *)y, desc->N, desc->C, desc->K);
        return check_launch();
    }
    const nsk_conv_desc_t c = linear_as_conv(desc);
    TAIL_TRY(nsk_conv2d_fwd(&c, x, w, y, workspace, workspace_bytes, stream));
    if (bias) {
        const long total = (long)desc->N * desc->K;
        const dim3 grid(stream_grid((size_t)total));
        if (desc->dtype == NSK_BF16)
            hipLaunchKernelGGL(add_bias_kernel<bf16_t>, grid, dim3(256), 0, (hipStream_t)stream, (bf16_t *)y, bias, total, desc->K);
        else
            hipLaunchKernelGGL(add_bias_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream, (float *)y, bias, total, desc->K);
        return check_launch();
    }
    return NSK_OK;
}

int nsk_linear_dgrad(const nsk_linear_desc_t *desc, const void *dy, const void *w, void *dx, int accumulate,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    TAIL_TRY(linear_check(desc));
    if (desc->N <= kSmallRows) {
        if (accumulate != 0 && accumulate != 1) return NSK_ERR_BAD_DESC;
        if (!dy || !w || !dx) return NSK_ERR_NULL;
        if (unaligned(dy) || unaligned(w) || unaligned(dx)) return NSK_ERR_ALIGNMENT;
        const dim3 grid((unsigned)((desc->C + 63) / 64), (unsigned)desc->N);
        if (desc->dtype == NSK_BF16)
            hipLaunchKernelGGL(linear_small_dgrad_kernel<bf16_t>, grid, dim3(256), 0, (hipStream_t)stream, (const bf16_t *)dy,
                               (const bf16_t *)w, (bf16_t *)dx, desc->N, desc->C, desc->K, accumulate);
        else
            hipLaunchKernelGGL(linear_small_dgrad_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream, (const float *)dy,
                               (const float *)w, (float *)dx, desc->N, desc->C, desc->K, accumulate);
        return check_launch();
    }
    const nsk_conv_desc_t c = linear_as_conv(desc);
    return nsk_conv2d_dgrad(&c, dy, w, dx, accumulate, workspace, workspace_bytes, stream);
}

int nsk_linear_wgrad(const nsk_linear_desc_t *desc, const void *x, const void *dy, float *dw, float *db, int accumulate,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    TAIL_TRY(linear_check(desc));
    if (db && unaligned(db)) return NSK_ERR_ALIGNMENT;
    const nsk_conv_desc_t c = linear_as_conv(desc);
    TAIL_TRY(nsk_conv2d_wgrad(&c, x, dy, dw, accumulate, workspace, workspace_bytes, stream));
    if (db) {
        // (the size query has room for the shares; a call with less than it asked for, but enough for dw, gets the one launch)
        if (bias_in_shares(desc) && workspace && workspace_bytes >= bias_share_bytes(desc) && !((uintptr_t)workspace & 15)) {
            const int rows = (desc->N + kBiasShares - 1) / kBiasShares, shares = (desc->N + rows - 1) / rows;
            const dim3 grid((unsigned)((desc->K + 63) / 64), (unsigned)shares);
            if (desc->dtype == NSK_BF16)
                hipLaunchKernelGGL(bias_partial_kernel<bf16_t>, grid, dim3(256), 0, (hipStream_t)stream, (const bf16_t *)dy, (float *)workspace, desc->N, desc->K, rows);
            else
                hipLaunchKernelGGL(bias_partial_kernel<float>, grid, dim3(256), 0, (hipStream_t)stream, (const float *)dy, (float *)workspace, desc->N, desc->K, rows);
            hipLaunchKernelGGL(bias_final_kernel, dim3((unsigned)((desc->K + 15) / 16)), dim3(64), 0, (hipStream_t)stream, (const float *)workspace, db, shares, desc->K, accumulate);
            return check_launch();
        }
#define NSK_BIAS(T, CB)                                                                                                  \
    hipLaunchKernelGGL((bias_grad_kernel<T, CB>), dim3((unsigned)((desc->K + CB - 1) / CB)), dim3(1024), 0, (hipStream_t)stream, \
                       (const T *)dy, db, desc->N, desc->K, accumulate)
        if (desc->dtype == NSK_BF16) {
            if (desc->N < 1024) NSK_BIAS(bf16_t, 64); else NSK_BIAS(bf16_t, 16);
        } else {
            if (desc->N < 1024) NSK_BIAS(float, 64); else NSK_BIAS(float, 16);
        }
#undef NSK_BIAS
        return check_launch();
    }
    return NSK_OK;
}

int nsk_transpose2d(int dtype, int rows, int cols, const void *src, void *dst, void *stream)
{
    if (rows <= 0 || cols <= 0 || !dtype_ok(dtype)) return NSK_ERR_BAD_DESC;
    if (!src || !dst) return NSK_ERR_NULL;
    if (unaligned(src) || unaligned(dst)) return NSK_ERR_ALIGNMENT;
    // [rows][cols] -> [cols][rows] is the NHWC -> NCHW copy of one image with rows pixels and cols channels
    return launch_nhwc_to_nchw(dtype, src, dst, 1, cols, rows, 1, 0, (hipStream_t)stream);
}

int nsk_softmax_xent_fwd(int dtype, int N, int K, const void *logits, const int *labels, float *per_sample, float *loss,
                         void *stream)
{
    if (N <= 0 || K <= 0 || !dtype_ok(dtype)) return NSK_ERR_BAD_DESC;
    if (!logits || !labels || !per_sample || !loss) return NSK_ERR_NULL;
    if (unaligned(logits) || unaligned(labels) || unaligned(per_sample) || unaligned(loss)) return NSK_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)((N + 3) / 4));
    if (dtype == NSK_BF16)
        hipLaunchKernelGGL((xent_kernel<bf16_t, 0>), grid, dim3(256), 0, st, (const bf16_t *)logits, labels, N, K, per_sample,
                           (bf16_t *)nullptr, 0.f);
    else
        hipLaunchKernelGGL((xent_kernel<float, 0>), grid, dim3(256), 0, st, (const float *)logits, labels, N, K, per_sample,
                           (float *)nullptr, 0.f);
    hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, st, per_sample, N, loss);
    return check_launch();
}

int nsk_softmax_xent_bwd(int dtype, int N, int K, const void *logits, const int *labels, float dloss, void *dlogits,
                         void *stream)
{
    if (N <= 0 || K <= 0 || !dtype_ok(dtype)) return NSK_ERR_BAD_DESC;
    if (!logits || !labels || !dlogits) return NSK_ERR_NULL;
    if (unaligned(logits) || unaligned(labels) || unaligned(dlogits)) return NSK_ERR_ALIGNMENT;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)((N + 3) / 4));
    const float coef = dloss / (float)N;
    if (dtype == NSK_BF16)
        hipLaunchKernelGGL((xent_kernel<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t *)logits, labels, N, K,
                           (float *)nullptr, (bf16_t *)dlogits, coef);
    else
        hipLaunchKernelGGL((xent_kernel<float, 1>), grid, dim3(256), 0, st, (const float *)logits, labels, N, K,
                           (float *)nullptr, (float *)dlogits, coef);
    return check_launch();
}

// Validates one parameter record and appends it to the launch table.
static int add_param(const nsk_param_t &q, bool adam, float wd_field, ParamTable *tab, int slot, size_t *max_n)
{
    if (q.n == 0) return NSK_ERR_BAD_DESC;
    if (!q.w || !q.grad || !q.state1 || (adam && !q.state2)) return NSK_ERR_NULL;
    if (unaligned(q.w) || unaligned(q.grad) || unaligned(q.state1) || (adam && unaligned(q.state2)) || (q.w_lp && unaligned(q.w_lp)))
        return NSK_ERR_ALIGNMENT;
    ParamEntry &e = tab->e[slot];
    e.w = q.w; e.g = q.grad; e.s1 = q.state1; e.s2 = adam ? q.state2 : nullptr;
    e.w_lp = (bf16_t *)q.w_lp;
    e.n = q.n;
    e.wd = wd_field;
    if (q.n > *max_n) *max_n = q.n;
    return NSK_OK;
}

static int optimizer_launch(bool adam, int count, const nsk_param_t *params, float lr, float momentum, AdamCoef ac,
                            const float *grad_scale, void *stream)
{
    if (count <= 0) return NSK_ERR_BAD_DESC;
    if (!params) return NSK_ERR_NULL;
    if (grad_scale && ((uintptr_t)grad_scale & 3)) return NSK_ERR_ALIGNMENT;
    // validate everything before the first launch
    for (int i = 0; i < count; ++i) {
        ParamTable scratch;
        size_t mx = 0;
        TAIL_TRY(add_param(params[i], adam, 0.f, &scratch, 0, &mx));
    }
    for (int base = 0; base < count; base += kMaxParams) {
        const int m = count - base < kMaxParams ? count - base : kMaxParams;
        ParamTable tab{};
        size_t max_n = 0;
        for (int i = 0; i < m; ++i) {
            const nsk_param_t &q = params[base + i];
            TAIL_TRY(add_param(q, adam, adam ? 1.f - lr * q.weight_decay : q.weight_decay, &tab, i, &max_n));
        }
        size_t bx = (max_n + 255) / 256;
        if (bx > 1024) bx = 1024;
        const dim3 grid((unsigned)bx, (unsigned)m);
        if (adam)
            hipLaunchKernelGGL(optimizer_kernel<true>, grid, dim3(256), 0, (hipStream_t)stream, tab, lr, 0.f, ac, grad_scale);
        else
            hipLaunchKernelGGL(optimizer_kernel<false>, grid, dim3(256), 0, (hipStream_t)stream, tab, lr, momentum, ac, grad_scale);
    }
    return check_launch();
}

int nsk_sgd_momentum_step_multi(int count, const nsk_param_t *params, float lr, float momentum, const float *grad_scale,
                                void *stream)
{
    return optimizer_launch(false, count, params, lr, momentum, AdamCoef{}, grad_scale, stream);
}

int nsk_adamw_step_multi(int count, const nsk_param_t *params, int step, float lr, float beta1, float beta2, float eps,
                         const float *grad_scale, void *stream)
{
    if (step < 1 || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f)) return NSK_ERR_BAD_DESC;
    AdamCoef ac;
    ac.lr = lr; ac.beta1 = beta1; ac.beta2 = beta2; ac.eps = eps;
    ac.c1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    ac.c2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    return optimizer_launch(true, count, params, lr, 0.f, ac, grad_scale, stream);
}

int nsk_sgd_momentum_step(size_t n, float *w, float *grad, float *velocity, void *w_lp, float lr, float momentum,
                          float weight_decay, const float *grad_scale, void *stream)
{
    const nsk_param_t p = {w, grad, velocity, nullptr, w_lp, n, weight_decay};
    return nsk_sgd_momentum_step_multi(1, &p, lr, momentum, grad_scale, stream);
}

int nsk_adamw_step(size_t n, float *w, float *grad, float *m, float *v, void *w_lp, int step, float lr, float beta1,
                   float beta2, float eps, float weight_decay, const float *grad_scale, void *stream)
{
    const nsk_param_t p = {w, grad, m, v, w_lp, n, weight_decay};
    return nsk_adamw_step_multi(1, &p, step, lr, beta1, beta2, eps, grad_scale, stream);
}

int nsk_sumsq_accumulate(size_t n, const float *g, float *partials, float *sumsq, void *stream)
{
    if (n == 0) return NSK_ERR_BAD_DESC;
    if (!g || !partials || !sumsq) return NSK_ERR_NULL;
    if (unaligned(g) || unaligned(partials) || ((uintptr_t)sumsq & 3)) return NSK_ERR_ALIGNMENT;
    size_t nb = (n + 1023) / 1024;
    if (nb > NSK_SUMSQ_PARTIALS) nb = NSK_SUMSQ_PARTIALS;
    hipLaunchKernelGGL(sumsq_partial_kernel, dim3((unsigned)nb), dim3(1024), 0, (hipStream_t)stream, n, g, partials);
    hipLaunchKernelGGL(sumsq_final_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, partials, (int)nb, sumsq);
    return check_launch();
}

int nsk_clip_scale_multi(int count, const float *const *g, const size_t *n, float max_norm, float *partials, float *sumsq, float *scale, void *stream)
{
    if (count <= 0 || !(max_norm > 0.f)) return NSK_ERR_BAD_DESC;
    if (!g || !n || !partials || !sumsq || !scale) return NSK_ERR_NULL;
    if (unaligned(partials) || ((uintptr_t)sumsq & 3) || ((uintptr_t)scale & 3)) return NSK_ERR_ALIGNMENT;
    size_t most = 0;
    for (int i = 0; i < count; ++i) {
        if (n[i] == 0) return NSK_ERR_BAD_DESC;
        if (!g[i]) return NSK_ERR_NULL;
        if (unaligned(g[i])) return NSK_ERR_ALIGNMENT;
        if (n[i] > most) most = n[i];
    }
    size_t nb = (most + 1023) / 1024;
    if (nb > NSK_SUMSQ_PARTIALS) nb = NSK_SUMSQ_PARTIALS;
    for (int at = 0; at < count; at += kMaxSumsq) {
        SumsqTable t{};
        t.count = count - at < kMaxSumsq ? count - at : kMaxSumsq;
        t.add = at > 0;
        for (int i = 0; i < t.count; ++i) {
            t.g[i] = g[at + i];
            t.n[i] = n[at + i];
        }
        hipLaunchKernelGGL(sumsq_multi_kernel, dim3((unsigned)nb), dim3(1024), 0, (hipStream_t)stream, t, partials);
    }
    hipLaunchKernelGGL(clip_final_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, partials, (int)nb, max_norm, sumsq, scale);
    return check_launch();
}

int nsk_clip_scale(const float *sumsq, float max_norm, float *scale, void *stream)
{
    if (!sumsq || !scale) return NSK_ERR_NULL;
    if (!(max_norm > 0.f)) return NSK_ERR_BAD_DESC;
    if (((uintptr_t)sumsq & 3) || ((uintptr_t)scale & 3)) return NSK_ERR_ALIGNMENT;
    hipLaunchKernelGGL(clip_scale_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, sumsq, max_norm, scale);
    return check_launch();
}

}  // extern "C"
