// Batch-norm (batch statistics) + residual add + ReLU, forward and backward, as HBM-streaming
// kernels.  The paper runs these element-wise steps unfused and names ReLU fusion as future work
// (conclusion); here each direction is one statistics pass and one fused apply pass:
//
//   forward : stats   x -> per-block partial sums          (read x)
//             finalize -> mean, invstd, scale, bias         (tiny)
//             apply   out = relu?(x*scale + bias [+ res])   (read x [,res], write out)
//   backward: reduce  dbeta, dgamma partials                (read x, out, dout)
//             finalize -> dbeta, dgamma, coefficients       (tiny)
//             apply   dx, dres                              (read x, out, dout; write dx [,dres])
//
// Statistics are accumulated in fp32 around a per-channel shift (the channel's first element), so
// E[(x-s)^2] - E[x-s]^2 does not cancel badly, and the per-block partials are combined in fp64 in
// a fixed order (reproducible, no atomics).
//
// Two code paths: a vectorised NHWC path (16-byte accesses, 8-byte ones in bf16 where C % 8 is 4; a
// thread keeps the same channels for all its rows) and a generic strided path that serves NCHW and
// channel counts that are not a multiple of four.
#include <algorithm>
#include <type_traits>

#include "nsk_internal.h"

namespace nsk {
namespace {

template <typename T, int V> using VecOf = T __attribute__((ext_vector_type(V)));

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Butterfly sum: every lane ends with the same value, combined in a fixed order.
__device__ inline double wave_sum_f64(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Channel counts whose vectors divide a block: the calls that hand a ReLU mask or an activation's coefficients from pass to
// pass take these.
bool nhwc_fast(const nsk_bn_desc_t &d)
{
    if (d.layout != NSK_NHWC) return false;
    const int VEC = d.dtype == NSK_BF16 ? 8 : 4;
    if (d.C % VEC) return false;
    const int cv = d.C / VEC;
    return cv <= 256 && 256 % cv == 0;
}

// Elements per access of the NHWC path, 0: the generic path, which is the faster one for small tensors of few channels (a block's
// last sums are longer here, the generic path divides per element).  Forward + backward with ReLU, 16 images, us, generic /
// here, thousands of elements: bf16 24 channels 198 16 / 19, 433 18 / 22, 693 24 / 23; 96 181 17 / 18, 433 21 / 22, 661 26 /
// 21; with 8-byte vectors 36 297 18 / 18, 441 19 / 19, 689 24 / 20; 100 189 17 / 19, 264 19 / 18, 400 21 / 18; fp32 12 300 17 /
// 20, 432 22 / 21; 24 198 17 / 19, 294 18 / 18, 433 23 / 20; 100 189 17 / 19, 264 19 / 18, 400 24 / 18.
int nhwc_vec(const nsk_bn_desc_t &d)
{
    if (d.layout != NSK_NHWC || d.C % 4) return 0;
    const int vec = d.dtype == NSK_BF16 && d.C % 8 == 0 ? 8 : 4;
    const long least = d.dtype == NSK_F32 ? (d.C < 16 ? 384L << 10 : 256L << 10) : vec == 4 && d.C >= 48 ? 256L << 10 : 512L << 10;
    return nhwc_fast(d) || (long)d.N * d.H * d.W * d.C >= least ? vec : 0;
}

// ----------------------------------------------------------------------------- NHWC path
// A block of 256 threads covers RP whole rows of the (up to 256) channel vectors of its chunk blockIdx.y: thread t has vector
// t % CV of row t / CV, and keeps it.  Where CV does not divide 256 the last 256 % CV threads idle, which costs less than the
// generic path's strided element accesses.  Measured with ReLU, 64 images of 28x28, forward, backward (us, generic / here):
// bf16 96 channels 39, 96 / 16, 25, 100 channels 38, 91 / 15, 28; fp32 100 channels 43, 105 / 18, 35; bf16 1000 channels, 7x7
// 36, 83 / 22, 29; 96 channels at 56x56 behind a convolution that left 3136 rows of sums 55, 358 / 25, 60.
struct Tile {
    int cv0, CV, RP, cv, rr;
    bool live;
};
template <int V> __device__ inline Tile tile_of(int C)
{
    Tile t;
    t.cv0 = blockIdx.y * 256;
    t.CV = min(C / V - t.cv0, 256);
    t.RP = 256 / t.CV;
    t.rr = threadIdx.x / t.CV;
    t.cv = threadIdx.x - t.rr * t.CV;
    t.live = t.rr < t.RP;
    t.cv += t.cv0;
    return t;
}

// Accumulates, per channel, sum(f0) and sum(f1) over the rows of this block, where (f0,f1) is
//   MODE 0 (forward stats):  (x - shift, (x - shift)^2)
//   MODE 1 (backward)     :  (dz, dz * xhat)
template <typename T, int VEC, int MODE>
__global__ __launch_bounds__(256) void bn_reduce_nhwc(const T *__restrict__ x, const T *__restrict__ out,
                                                      const T *__restrict__ dout, const float *__restrict__ mean,
                                                      const float *__restrict__ invstd, int relu, long M, int C,
                                                      long rows_per_block, float *__restrict__ p0,
                                                      float *__restrict__ p1, int noshift)
{
    typedef VecOf<T, VEC> Vec;
    const Tile t = tile_of<VEC>(C);
    const int cv = t.live ? t.cv : t.cv0, RP = t.RP;
    float s0[VEC], s1[VEC], sh[VEC], sc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        s0[e] = 0.f;
        s1[e] = 0.f;
        if (MODE == 0) {
            sh[e] = noshift ? 0.f : (float)x[cv * VEC + e];
            sc[e] = 1.f;
        } else {
            sh[e] = mean[cv * VEC + e];
            sc[e] = invstd[cv * VEC + e];
        }
    }
    const long r_begin = (long)blockIdx.x * rows_per_block;
    const long r_end = t.live ? min(M, r_begin + rows_per_block) : 0;
#pragma unroll 4
    for (long r = r_begin + t.rr; r < r_end; r += RP) {
        const long off = r * C + cv * VEC;
        const Vec xv = *(const Vec *)(x + off);
        if (MODE == 0) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float dlt = (float)xv[e] - sh[e];
                s0[e] += dlt;
                s1[e] += dlt * dlt;
            }
        } else {
            const Vec gv = *(const Vec *)(dout + off);
            Vec ov;
            if (relu) ov = *(const Vec *)(out + off);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                float dz = (float)gv[e];
                if (relu && !((float)ov[e] > 0.f)) dz = 0.f;
                s0[e] += dz;
                s1[e] += dz * (((float)xv[e] - sh[e]) * sc[e]);
            }
        }
    }
    __shared__ __attribute__((aligned(16))) float red0[256 * VEC], red1[256 * VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        red0[threadIdx.x * VEC + e] = s0[e];
        red1[threadIdx.x * VEC + e] = s1[e];
    }
    __syncthreads();
    // The columns of the chunk are summed over the RP row groups (row group rr holds its channels at rr*CC..).  Few channels make RP
    // large (85 for 24 channels in bf16): up to 16 threads a column then take every 16th group each, and all is added in
    // fp64.  With one thread and one float chain a column that chain was the largest error of the pass (24 channels, 62
    // images of 12x16: invstd 1.5e-7, dgamma 2.0e-7 against 64 bits) and took longer (16 channels, 256 images of 32x32,
    // forward and backward 14.2, 20.5 -> 13.2, 19.8 us).
    const int CC = t.CV * VEC, c0 = t.cv0 * VEC;
    if (RP > 32) {          // (CC is at most 56)
        const int parts = min(256 / CC, 16), q = threadIdx.x / CC, c = threadIdx.x - q * CC;
        double a0 = 0., a1 = 0.;
        if (q < parts)
            for (int g = q; g < RP; g += parts) {
                a0 += red0[g * CC + c];
                a1 += red1[g * CC + c];
            }
        __syncthreads();
        double *const few0 = (double *)red0, *const few1 = (double *)red1;
        if (q < parts) {
            few0[q * CC + c] = a0;
            few1[q * CC + c] = a1;
        }
        __syncthreads();
        if (q == 0) {
            for (int g = 1; g < parts; ++g) {
                a0 += few0[g * CC + c];
                a1 += few1[g * CC + c];
            }
            p0[(long)blockIdx.x * C + c0 + c] = (float)a0;
            p1[(long)blockIdx.x * C + c0 + c] = (float)a1;
        }
        return;
    }
    for (int c = threadIdx.x; c < CC; c += 256) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll 8
        for (int g = 0; g < RP; ++g) {
            a0 += red0[g * CC + c];
            a1 += red1[g * CC + c];
        }
        p0[(long)blockIdx.x * C + c0 + c] = a0;
        p1[(long)blockIdx.x * C + c0 + c] = a1;
    }
}

template <typename T, int VEC, bool HAS_RES, bool RELU>
__global__ __launch_bounds__(256) void bn_apply_nhwc(const T *__restrict__ x, const T *__restrict__ res,
                                                     T *__restrict__ out, const float *__restrict__ scale,
                                                     const float *__restrict__ bias, long nvec, int C,
                                                     unsigned char *__restrict__ mask)
{
    typedef VecOf<T, VEC> Vec;
    // a thread always sees the same VEC channels: their coefficients live in registers
    const Tile t = tile_of<VEC>(C);
    if (!t.live) return;
    const int c0 = t.cv * VEC, CV = C / VEC;
    float sc[VEC], bi[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        sc[e] = scale[c0 + e];
        bi[e] = bias[c0 + e];
    }
    for (long i = ((long)blockIdx.x * t.RP + t.rr) * CV + t.cv; i < nvec; i += (long)gridDim.x * t.RP * CV) {
        const Vec xv = __builtin_nontemporal_load((const Vec *)(x + i * VEC));
        Vec rv;
        if (HAS_RES) rv = __builtin_nontemporal_load((const Vec *)(res + i * VEC));
        Vec ov;
        unsigned bits = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float z = (float)xv[e] * sc[e] + bi[e];
            if (HAS_RES) z += (float)rv[e];
            if (RELU) z = z > 0.f ? z : 0.f;
            ov[e] = (T)z;
            bits |= ((float)ov[e] > 0.f ? 1u : 0u) << e;   // of the value as stored
        }
        __builtin_nontemporal_store(ov, (Vec *)(out + i * VEC));
        if (RELU && mask) mask[i] = (unsigned char)bits;
    }
}

// dx = a*(dz - b - xhat*cc) with a = gamma*invstd, b = dbeta/M, cc = dgamma/M ; dres = dz
// RELU: 0 none, 1 with the mask of the reduction or forward pass, 2 from the sign of out
template <typename T, int VEC, bool HAS_RES, int RELU>
__global__ __launch_bounds__(256) void bn_bwd_apply_nhwc(const T *__restrict__ x, const T *__restrict__ out,
                                                         const T *__restrict__ dout, T *__restrict__ dx,
                                                         T *__restrict__ dres, const float *__restrict__ mean,
                                                         const float *__restrict__ invstd,
                                                         const float *__restrict__ coef, long nvec, int C,
                                                         const unsigned char *__restrict__ mask)
{
    typedef VecOf<T, VEC> Vec;
    const Tile t = tile_of<VEC>(C);
    if (!t.live) return;
    const int c0 = t.cv * VEC, CV = C / VEC;   // fixed per thread, see bn_apply_nhwc
    float mu[VEC], is[VEC], ka[VEC], kb[VEC], kc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        mu[e] = mean[c0 + e];
        is[e] = invstd[c0 + e];
        ka[e] = coef[c0 + e];
        kb[e] = coef[C + c0 + e];
        kc[e] = coef[2 * C + c0 + e];
    }
    for (long i = ((long)blockIdx.x * t.RP + t.rr) * CV + t.cv; i < nvec; i += (long)gridDim.x * t.RP * CV) {
        const Vec xv = __builtin_nontemporal_load((const Vec *)(x + i * VEC));
        const Vec gv = __builtin_nontemporal_load((const Vec *)(dout + i * VEC));
        // ReLU mask of these VEC elements, written by the reduction pass (bit e set: out > 0)
        unsigned bits = ~0u;
        if (RELU == 1) bits = __builtin_nontemporal_load(mask + i);
        if (RELU == 2) {
            const Vec ov = __builtin_nontemporal_load((const Vec *)(out + i * VEC));
            bits = 0;
#pragma unroll
            for (int e = 0; e < VEC; ++e) bits |= ((float)ov[e] > 0.f ? 1u : 0u) << e;
        }
        Vec dxv, drv;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float dz = (float)gv[e];
            if (RELU && !((bits >> e) & 1u)) dz = 0.f;
            const float xhat = ((float)xv[e] - mu[e]) * is[e];
            dxv[e] = (T)(ka[e] * (dz - kb[e] - xhat * kc[e]));
            drv[e] = (T)dz;
        }
        __builtin_nontemporal_store(dxv, (Vec *)(dx + i * VEC));
        if (HAS_RES) __builtin_nontemporal_store(drv, (Vec *)(dres + i * VEC));
    }
}

// ----------------------------------------------------------------------------- NHWC path, channel counts of nhwc_fast
// The sums: a block has a chunk of at most 128 channels (64 up to 128 channels: at least 128 bytes of a row) and whole row groups of
// it, 1024 threads, sixteen wavefronts a CU with four rows each on their way.  256 blocks then leave 256/chunks rows of sums in all,
// 131 KB at 64 channels, 8 KB at 1024, where 512 blocks over whole rows left 2 * 512 * C floats (4 MB at 1024 channels, which
// the next launch read column by column).  That makes it cheap to finish the sums in the apply pass, block by block, without the
// launch between (4-5 us behind a busy one, for next to no work).
// Measured, us, before / now, bf16, statistics + apply of one direction: 64 images of 7x7x512 backward 15.2 / 10.4, 28x28x128
// 23.8 / 19.4, 256 images of 16x16x32 14.2 / 10.6; 128 images of 14x14x1024 58.2 / 51, without a mask 82 / 67, forward with its own
// statistics 55 / 43; 64 images of 112x112x64 without a mask 157 / 138.
constexpr int kBnThreads = 1024, kBnChunk = 128;      // (a chunk has 64 channels up to 128 channels)
struct Chunk {
    int c0, CC, CV, RP, cv, rr;    // first channel and channels of the chunk, its vectors, rows at a time; this thread's vector and row
};
template <int VEC, int THREADS = kBnThreads> __device__ inline Chunk chunk_of(int C)
{
    Chunk k;
    k.CC = min(C, C > 128 ? kBnChunk : 64);
    k.c0 = blockIdx.y * k.CC;
    k.CV = k.CC / VEC;             // (a power of two)
    const int sh = __builtin_ctz(k.CV);
    k.RP = THREADS >> sh;
    k.rr = threadIdx.x >> sh;
    k.cv = threadIdx.x & (k.CV - 1);
    return k;
}

// Rows of a block: r = first + rr, first + rr + step, ... < end.  XCD: eighth e of the rows goes to the blocks that run on XCD e (blocks go to
// the eight in turn, and gridDim.x is a multiple of eight), in the sums and in the apply pass, so that what the sums have read of a tensor is
// still in that XCD's L2; the pipelined convolution kernels hand out their tiles alike.  Else the sums take their rows in one piece, the apply
// pass in turn.  Backward, both passes, bf16, 64 images of 28x28x128 (12.8 MB each of x and dout) 18.4 -> 13.9 us.
struct Walk {
    long first, end, step;
};
template <bool XCD> __device__ inline Walk walk_rows(long M, int per)
{
    if (!XCD) return {(long)blockIdx.x * per, M, (long)gridDim.x * per};
    const long share = (M + 7) >> 3, start = (long)(blockIdx.x & 7) * share;
    return {start + (long)(blockIdx.x >> 3) * per, min(M, start + share), (long)(gridDim.x >> 3) * per};
}

// buf[g][o], g < n groups, o < W columns (n * W = `slots` threads' worth, both powers of two) -> buf[0][o], eight groups at a time, fixed order
__device__ inline void fold_groups(double *buf, int n, int W)      // (n * W / 8 is at most the threads of the block)
{
    while (n > 1) {
        const int m = n > 8 ? n / 8 : 1, per = n / m;
        double v = 0.;
        __syncthreads();
        const int o = threadIdx.x & (W - 1);
        // (more columns than threads never: W is at most 2 * kBnChunk)
        const int j = threadIdx.x / W;
        if (j < m)
            for (int i = 0; i < per; ++i) v += buf[(size_t)(j + i * m) * W + o];
        __syncthreads();
        if (j < m) buf[(size_t)j * W + o] = v;
        n = m;
    }
    __syncthreads();
}

// Sums over G rows of partial sums, of CC channels from c0 on: lds[c] and lds[CC + c].  `lds` holds 4 * THREADS doubles.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
template <int THREADS>
__device__ inline void chunk_sums(const float *__restrict__ p0, const float *__restrict__ p1, int G, int C, int c0, int CC, double *lds)
{
    const int W = CC / 2, col = threadIdx.x & (W - 1), groups = THREADS / W, half = W / 2;     // four channels a thread
    const float *p = (col < half ? p0 : p1) + c0 + 4 * (col & (half - 1));
    double s[4] = {};
    const int g0 = threadIdx.x / W;
    int g = g0;
    for (; g + 3 * groups < G; g += 4 * groups) {
        f32x4_u v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const f32x4_u *)(p + (size_t)(g + i * groups) * C);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += ((double)v[0][e] + (double)v[1][e]) + ((double)v[2][e] + (double)v[3][e]);
    }
    for (; g < G; g += groups) {
        const f32x4_u v = *(const f32x4_u *)(p + (size_t)g * C);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += (double)v[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) lds[(size_t)g0 * 4 * W + 4 * col + e] = s[e];
    fold_groups(lds, groups, 4 * W);
}

// As bn_reduce_nhwc: per channel sum(f0) and sum(f1) over the rows of this block.  The ReLU mask of the backward pass is one byte per
// vector: read (mask_in), or found from `out` (MODE 1) or from the coefficients `act` of an activation that was never stored (2), and kept.
template <typename T, int VEC, int MODE, int THREADS, bool XCD>
__global__ __launch_bounds__(THREADS) void bn_sums_fast(const T *__restrict__ x, const T *__restrict__ out, const T *__restrict__ dout,
                                                           const float *__restrict__ mean, const float *__restrict__ invstd, int relu,
                                                           long M, int C, long rows_per_block, float *__restrict__ p0, float *__restrict__ p1,
                                                           unsigned char *__restrict__ mask, const unsigned char *__restrict__ mask_in,
                                                           const float *__restrict__ act, float *__restrict__ shift)
{
    typedef VecOf<T, VEC> Vec;
    const Chunk k = chunk_of<VEC, THREADS>(C);
    const int ch = k.c0 + k.cv * VEC;
    float s0[VEC], s1[VEC], sh[VEC], sc[VEC], as[VEC], ab[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        s0[e] = 0.f;
        s1[e] = 0.f;
        as[e] = MODE == 2 ? act[ch + e] : 0.f;
        ab[e] = MODE == 2 ? act[C + ch + e] : 0.f;
        sh[e] = MODE == 0 ? (float)x[ch + e] : mean[ch + e];
        sc[e] = MODE == 0 ? 1.f : invstd[ch + e];
        // (the apply pass needs it in every block, and may be overwriting x)
        if (MODE == 0 && blockIdx.x == 0 && k.rr == 0) shift[ch + e] = sh[e];
    }
    const Walk w = XCD ? walk_rows<true>(M, k.RP)
                       : Walk{(long)blockIdx.x * rows_per_block, min(M, (long)(blockIdx.x + 1) * rows_per_block), k.RP};
    const long step = XCD ? w.step : k.RP;
    if constexpr (MODE == 0) {
        // two chains, every other row each: beyond 16 M elements, where blocks of 256 threads would have been 2048, one chain would be twice as
        // long as theirs (invstd of 128 images of 112x112x128, bf16, against 64 bits: 2.9e-7 with one chain, 1.2e-7 with two, as with those blocks)
        float t0[VEC] = {}, t1[VEC] = {};
        auto add = [&](const Vec xv, float (&a)[VEC], float (&b)[VEC]) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float dlt = (float)xv[e] - sh[e];
                a[e] += dlt;
                b[e] += dlt * dlt;
            }
        };
        long r = w.first + k.rr;
#pragma unroll 2
        for (; r + step < w.end; r += 2 * step) {
            const Vec even = *(const Vec *)(x + r * C + ch), odd = *(const Vec *)(x + (r + step) * C + ch);
            add(even, s0, s1);
            add(odd, t0, t1);
        }
        if (r < w.end) add(*(const Vec *)(x + r * C + ch), s0, s1);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            s0[e] += t0[e];
            s1[e] += t1[e];
        }
    } else {
#pragma unroll 4
        for (long r = w.first + k.rr; r < w.end; r += step) {
            const long off = r * C + ch;
            const Vec xv = *(const Vec *)(x + off), gv = *(const Vec *)(dout + off);
            unsigned bits = 0;
            if (MODE == 1 && mask_in) {
                bits = mask_in[off / VEC];
            } else if (MODE == 2) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) bits |= ((float)(T)((float)xv[e] * as[e] + ab[e]) > 0.f ? 1u : 0u) << e;
                mask[off / VEC] = (unsigned char)bits;
            } else if (relu) {
                const Vec ov = *(const Vec *)(out + off);
#pragma unroll
                for (int e = 0; e < VEC; ++e) bits |= ((float)ov[e] > 0.f ? 1u : 0u) << e;
                mask[off / VEC] = (unsigned char)bits;
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                float dz = (float)gv[e];
                if ((MODE == 2 || relu) && !((bits >> e) & 1u)) dz = 0.f;
                s0[e] += dz;
                s1[e] += dz * (((float)xv[e] - sh[e]) * sc[e]);
            }
        }
    }
    // the RP row groups of a channel are added in fp64
    extern __shared__ __attribute__((aligned(16))) float red[];      // [RP][2 * CC]
    float *const mine = red + (size_t)k.rr * 2 * k.CC + k.cv * VEC;
#pragma unroll
    for (int e = 0; e < VEC; e += 4) {
        *(f32x4 *)(mine + e) = f32x4{s0[e], s0[e + 1], s0[e + 2], s0[e + 3]};
        *(f32x4 *)(mine + k.CC + e) = f32x4{s1[e], s1[e + 1], s1[e + 2], s1[e + 3]};
    }
    __syncthreads();
    const int W = 2 * k.CC, o = threadIdx.x & (W - 1), n = THREADS / W;      // n partial columns of RP / n row groups each
    double v = 0.;
    for (int g = threadIdx.x / W; g < k.RP; g += n) v += (double)red[(size_t)g * W + o];
    __syncthreads();
    double *const d = (double *)red;
    d[threadIdx.x] = v;                // [n][W]
    fold_groups(d, n, W);
    if (threadIdx.x < W) (o < k.CC ? p0 : p1)[(long)blockIdx.x * C + k.c0 + (o & (k.CC - 1))] = (float)d[o];
}

struct BnFwdFinish {
    const float *p0, *p1, *gamma, *beta, *shift;       // shift: the sums are of x - shift (nullptr: of x)
    float *save_mean, *save_invstd, *running_mean, *running_var;
    double M;
    float eps, momentum;
    int G;
};
// From the sums of channel c: the coefficients of the apply pass and, from one block, what the call returns
__device__ inline void finish_fwd(const BnFwdFinish &f, int c, double S, double Q, bool write, float *scale, float *bias)
{
    const double ms = S / f.M;
    double var = Q / f.M - ms * ms;
    if (var < 0.0) var = 0.0;
    const double mean = (f.shift ? (double)f.shift[c] : 0.0) + ms;
    const double invstd = 1.0 / sqrt(var + (double)f.eps);
    const double sc = (double)f.gamma[c] * invstd;
    *scale = (float)sc;
    *bias = (float)((double)f.beta[c] - mean * sc);
    if (!write) return;
    f.save_mean[c] = (float)mean;
    f.save_invstd[c] = (float)invstd;
    if (f.running_mean) {
        const double unbiased = f.M > 1.0 ? var * f.M / (f.M - 1.0) : var;
        f.running_mean[c] = (float)((1.0 - (double)f.momentum) * (double)f.running_mean[c] + (double)f.momentum * mean);
        f.running_var[c] = (float)((1.0 - (double)f.momentum) * (double)f.running_var[c] + (double)f.momentum * unbiased);
    }
}

template <typename T, int VEC, bool HAS_RES, bool RELU, bool XCD>
__global__ __launch_bounds__(kBnThreads) void bn_apply_fast(const T *__restrict__ x, const T *__restrict__ res, T *__restrict__ out, long M,
                                                            int C, unsigned char *__restrict__ mask, const BnFwdFinish f)
{
    typedef VecOf<T, VEC> Vec;
    __shared__ double sums[4 * kBnThreads];
    __shared__ float coef[2][kBnChunk];
    const Chunk k = chunk_of<VEC>(C);
    chunk_sums<kBnThreads>(f.p0, f.p1, f.G, C, k.c0, k.CC, sums);
    if ((int)threadIdx.x < k.CC)
        finish_fwd(f, k.c0 + threadIdx.x, sums[threadIdx.x], sums[k.CC + threadIdx.x], blockIdx.x == 0, &coef[0][threadIdx.x], &coef[1][threadIdx.x]);
    __syncthreads();
    float sc[VEC], bi[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        sc[e] = coef[0][k.cv * VEC + e];
        bi[e] = coef[1][k.cv * VEC + e];
    }
    const Walk w = walk_rows<XCD>(M, k.RP);
#pragma unroll 2
    for (long r = w.first + k.rr; r < w.end; r += w.step) {
        const long off = r * C + k.c0 + k.cv * VEC;
        const Vec xv = __builtin_nontemporal_load((const Vec *)(x + off));
        Vec rv;
        if (HAS_RES) rv = __builtin_nontemporal_load((const Vec *)(res + off));
        Vec ov;
        unsigned bits = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float z = (float)xv[e] * sc[e] + bi[e];
            if (HAS_RES) z += (float)rv[e];
            if (RELU) z = z > 0.f ? z : 0.f;
            ov[e] = (T)z;
            bits |= ((float)ov[e] > 0.f ? 1u : 0u) << e;   // of the value as stored
        }
        __builtin_nontemporal_store(ov, (Vec *)(out + off));
        if (RELU && mask) mask[off / VEC] = (unsigned char)bits;
    }
}

struct BnBwdFinish {
    const float *p0, *p1, *gamma, *mean, *invstd;
    float *dgamma, *dbeta;
    double M;
    int G;
};

// dx = a*(dz - b - xhat*cc) with a = gamma*invstd, b = dbeta/M, cc = dgamma/M ; dres = dz
template <typename T, int VEC, bool HAS_RES, bool RELU, bool XCD>
__global__ __launch_bounds__(kBnThreads) void bn_bwd_apply_fast(const T *__restrict__ x, const T *__restrict__ dout, T *__restrict__ dx,
                                                                T *__restrict__ dres, long M, int C, const unsigned char *__restrict__ mask,
                                                                const BnBwdFinish f)
{
    typedef VecOf<T, VEC> Vec;
    __shared__ double sums[4 * kBnThreads];
    __shared__ float coef[5][kBnChunk];
    const Chunk k = chunk_of<VEC>(C);
    chunk_sums<kBnThreads>(f.p0, f.p1, f.G, C, k.c0, k.CC, sums);
    if ((int)threadIdx.x < k.CC) {
        const int c = k.c0 + threadIdx.x;
        const double S = sums[threadIdx.x], Q = sums[k.CC + threadIdx.x];
        if (blockIdx.x == 0) {
            f.dbeta[c] = (float)S;
            f.dgamma[c] = (float)Q;
        }
        coef[0][threadIdx.x] = f.mean[c];
        coef[1][threadIdx.x] = f.invstd[c];
        coef[2][threadIdx.x] = f.gamma[c] * f.invstd[c];
        coef[3][threadIdx.x] = (float)(S / f.M);
        coef[4][threadIdx.x] = (float)(Q / f.M);
    }
    __syncthreads();
    float mu[VEC], is[VEC], ka[VEC], kb[VEC], kc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const int c = k.cv * VEC + e;
        mu[e] = coef[0][c];
        is[e] = coef[1][c];
        ka[e] = coef[2][c];
        kb[e] = coef[3][c];
        kc[e] = coef[4][c];
    }
    const Walk w = walk_rows<XCD>(M, k.RP);
#pragma unroll 2
    for (long r = w.first + k.rr; r < w.end; r += w.step) {
        const long off = r * C + k.c0 + k.cv * VEC;
        const Vec xv = __builtin_nontemporal_load((const Vec *)(x + off));
        const Vec gv = __builtin_nontemporal_load((const Vec *)(dout + off));
        const unsigned bits = RELU ? __builtin_nontemporal_load(mask + off / VEC) : ~0u;
        Vec dxv, drv;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float dz = (float)gv[e];
            if (RELU && !((bits >> e) & 1u)) dz = 0.f;
            const float xhat = ((float)xv[e] - mu[e]) * is[e];
            dxv[e] = (T)(ka[e] * (dz - kb[e] - xhat * kc[e]));
            drv[e] = (T)dz;
        }
        __builtin_nontemporal_store(dxv, (Vec *)(dx + off));
        if (HAS_RES) __builtin_nontemporal_store(drv, (Vec *)(dres + off));
    }
}

// ----------------------------------------------------------------------------- generic strided path
// element (n, c, s) lives at n*sn + c*sc + s*ss ; block (c, g) covers images [g*npg, (g+1)*npg)
template <typename T, int MODE>
__global__ __launch_bounds__(256) void bn_reduce_generic(const T *__restrict__ x, const T *__restrict__ out,
                                                         const T *__restrict__ dout, const float *__restrict__ mean,
                                                         const float *__restrict__ invstd, int relu, int N, long HW,
                                                         long sn, long scs, long ss, int npg, int C,
                                                         float *__restrict__ p0, float *__restrict__ p1, int noshift = 0)
{
    const int c = blockIdx.x, g = blockIdx.y;
    const float sh = MODE == 0 ? (noshift ? 0.f : (float)x[c * scs]) : mean[c];
    const float scl = MODE == 0 ? 1.f : invstd[c];
    float s0 = 0.f, s1 = 0.f;
    const int n_end = min(N, (g + 1) * npg);
    for (int n = g * npg; n < n_end; ++n)
        for (long s = threadIdx.x; s < HW; s += 256) {
            const long off = n * sn + c * scs + s * ss;
            if (MODE == 0) {
                const float dlt = (float)x[off] - sh;
                s0 += dlt;
                s1 += dlt * dlt;
            } else {
                float dz = (float)dout[off];
                if (relu && !((float)out[off] > 0.f)) dz = 0.f;
                s0 += dz;
                s1 += dz * (((float)x[off] - sh) * scl);
            }
        }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    __shared__ float w0[4], w1[4];
    if ((threadIdx.x & 63) == 0) {
        w0[threadIdx.x >> 6] = s0;
        w1[threadIdx.x >> 6] = s1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        p0[(long)g * C + c] = (w0[0] + w0[1]) + (w0[2] + w0[3]);
        p1[(long)g * C + c] = (w1[0] + w1[1]) + (w1[2] + w1[3]);
    }
}

template <typename T, bool NCHW>
__global__ __launch_bounds__(256) void bn_apply_generic(const T *__restrict__ x, const T *__restrict__ res,
                                                        T *__restrict__ out, const float *__restrict__ scale,
                                                        const float *__restrict__ bias, long total, int C, long HW,
                                                        int relu)
{
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int c = NCHW ? (int)((i / HW) % C) : (int)(i % C);
        float z = (float)x[i] * scale[c] + bias[c];
        if (res) z += (float)res[i];
        if (relu) z = z > 0.f ? z : 0.f;
        out[i] = (T)z;
    }
}

template <typename T, bool NCHW>
__global__ __launch_bounds__(256) void bn_bwd_apply_generic(const T *__restrict__ x, const T *__restrict__ out,
                                                            const T *__restrict__ dout, T *__restrict__ dx,
                                                            T *__restrict__ dres, const float *__restrict__ mean,
                                                            const float *__restrict__ invstd,
                                                            const float *__restrict__ coef, long total, int C,
                                                            long HW, int relu)
{
    const float *ca = coef, *cb = coef + C, *cc = coef + 2 * C;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int c = NCHW ? (int)((i / HW) % C) : (int)(i % C);
        float dz = (float)dout[i];
        if (relu && !((float)out[i] > 0.f)) dz = 0.f;
        const float xhat = ((float)x[i] - mean[c]) * invstd[c];
        dx[i] = (T)(ca[c] * (dz - cb[c] - xhat * cc[c]));
        if (dres) dres[i] = (T)dz;
    }
}

// Folds many rows of partial sums into few: out[j][c] = sum of in[r][c] over the j-th run of `run` rows, for the
// two arrays (sums, sums of squares) that follow each other in both buffers.  Fixed order: reproducible.
__global__ __launch_bounds__(256) void bn_stats_fold(const float *__restrict__ in, int R, int C, int run,
                                                     float *__restrict__ out, int R2)
{
    const int j = blockIdx.x;
    const int r0 = j * run, r1 = min(R, r0 + run);
    for (int c = blockIdx.y * 256 + threadIdx.x; c < 2 * C; c += gridDim.y * 256) {
        const int arr = c / C, cc = c - arr * C;
        const float *p = in + (size_t)arr * R * C + cc;
        // fp64: in float a share of 1500 rows would cost E[x^2] - E[x]^2 its last digits; eight loads on their way
        double s[4] = {};
        int r = r0;
        for (; r + 7 < r1; r += 8) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = p[(size_t)(r + e) * C];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += (double)v[e] + (double)v[e + 4];
        }
        for (; r < r1; ++r) s[0] += (double)p[(size_t)r * C];
        out[(size_t)arr * R2 * C + (size_t)j * C + cc] = (float)((s[0] + s[1]) + (s[2] + s[3]));
    }
}

// ----------------------------------------------------------------------------- finalize (tiny)
// Column sums of the two arrays of partial sums for channel c, by one block of 256 threads: every thread adds the
// rows g = t, t + 256, ... (four independent loads at a time), then lanes and wavefronts are combined in a fixed
// order.  The result is valid in thread 0.
__device__ inline void block_column_sums(const float *__restrict__ p0, const float *__restrict__ p1, int G, int C, int c,
                                         double *S_out, double *Q_out)
{
    __shared__ double part[2][4];
    const int t = threadIdx.x;
    double S = 0.0, Q = 0.0;
    int g = t;
    for (; g + 768 < G; g += 1024) {
        const float a0 = p0[(long)g * C + c], a1 = p0[(long)(g + 256) * C + c], a2 = p0[(long)(g + 512) * C + c],
                    a3 = p0[(long)(g + 768) * C + c];
        const float b0 = p1[(long)g * C + c], b1 = p1[(long)(g + 256) * C + c], b2 = p1[(long)(g + 512) * C + c],
                    b3 = p1[(long)(g + 768) * C + c];
        S += ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
        Q += ((double)b0 + (double)b1) + ((double)b2 + (double)b3);
    }
    for (; g < G; g += 256) {
        S += (double)p0[(long)g * C + c];
        Q += (double)p1[(long)g * C + c];
    }
    S = wave_sum_f64(S);
    Q = wave_sum_f64(Q);
    if ((t & 63) == 0) {
        part[0][t >> 6] = S;
        part[1][t >> 6] = Q;
    }
    __syncthreads();
    *S_out = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
    *Q_out = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
}

template <typename T>
__global__ __launch_bounds__(256) void bn_fwd_finalize(const float *__restrict__ p0, const float *__restrict__ p1, int G, int C, double M,
                                const T *__restrict__ x, long shift_stride, const float *__restrict__ gamma,
                                const float *__restrict__ beta, float eps, float momentum,
                                float *__restrict__ save_mean, float *__restrict__ save_invstd,
                                float *__restrict__ running_mean, float *__restrict__ running_var,
                                float *__restrict__ scale, float *__restrict__ bias)
{
    const int c = blockIdx.x;
    double S, Q;
    block_column_sums(p0, p1, G, C, c, &S, &Q);
    if (threadIdx.x != 0) return;
    const double ms = S / M;
    double var = Q / M - ms * ms;
    if (var < 0.0) var = 0.0;
    const double mean = (x ? (double)(float)x[c * shift_stride] : 0.0) + ms;   // x == nullptr: the sums are not shifted
    const double invstd = 1.0 / sqrt(var + (double)eps);
    save_mean[c] = (float)mean;
    save_invstd[c] = (float)invstd;
    const double sc = (double)gamma[c] * invstd;
    scale[c] = (float)sc;
    bias[c] = (float)((double)beta[c] - mean * sc);
    if (running_mean) {
        const double unbiased = M > 1.0 ? var * M / (M - 1.0) : var;
        running_mean[c] = (float)((1.0 - (double)momentum) * (double)running_mean[c] + (double)momentum * mean);
        running_var[c] = (float)((1.0 - (double)momentum) * (double)running_var[c] + (double)momentum * unbiased);
    }
}

__global__ __launch_bounds__(256) void bn_bwd_finalize(const float *__restrict__ p0, const float *__restrict__ p1, int G, int C, double M,
                                const float *__restrict__ gamma, const float *__restrict__ invstd,
                                float *__restrict__ dgamma, float *__restrict__ dbeta, float *__restrict__ coef)
{
    const int c = blockIdx.x;
    double S, Q;
    block_column_sums(p0, p1, G, C, c, &S, &Q);
    if (threadIdx.x != 0) return;
    dbeta[c] = (float)S;
    dgamma[c] = (float)Q;
    coef[c] = gamma[c] * invstd[c];
    coef[C + c] = (float)(S / M);
    coef[2 * C + c] = (float)(Q / M);
}

struct Geom {
    long M, HW, total;
    int G;
    int vec;              // NHWC path: elements per access (0: generic path)
    int chunks, RP;       // NHWC path: chunks of 256 vectors in a row, rows a block covers at a time
    long rows_per_block;
    int npg;              // generic path: images per partial block
    long sn, sc, ss;
};

Geom geometry(const nsk_bn_desc_t &d, bool backward)
{
    Geom g;
    g.HW = (long)d.H * d.W;
    g.M = (long)d.N * g.HW;
    g.total = g.M * d.C;
    g.vec = nhwc_vec(d);
    if (g.vec) {
        const int cv = d.C / g.vec, RP = cv < 256 ? 256 / cv : 1;
        g.chunks = ceil_div(cv, 256);
        g.RP = RP;
        // at least four passes of its 256 threads per block (measured on the 2-8 MB tensors of the CIFAR-sized network:
        // eight passes leave one block per CU there and the whole step 1.5% slower; two are no better than four)
        long G = (g.M + (long)RP * 4 - 1) / ((long)RP * 4);
        // few rows: one pass, while that makes no more than 64 blocks (bf16 64 channels, 4 images of 28x28, backward 12.7 -> 10.7)
        if (G < 64) G = (g.M + RP - 1) / RP < 64 ? (g.M + RP - 1) / RP : 64;
        // Measured: the forward statistics pass over a large tensor (one input stream) is fastest with eight blocks
        // per CU, the backward pass (three input streams) and small tensors with two.
        // More blocks also mean more partial sums for the finalize kernel to read (G x C floats, twice): the larger
        // count is only used while that stays within 2 MB per array.
        long cap = (!backward && g.total >= (16L << 20)) ? 2048 : 512;
        if (cap * d.C > (512L << 10)) cap = 512;
        // (other channel counts, up to 65535, stay within 2 MB per array throughout)
        if (!nhwc_fast(d) && cap * d.C > (512L << 10)) cap = (512L << 10) / d.C;
        if (G > cap) G = cap;
        if (G < 1) G = 1;
        g.rows_per_block = (g.M + G - 1) / G;
        g.G = (int)((g.M + g.rows_per_block - 1) / g.rows_per_block);
        g.npg = 0;
    } else {
        int G = 1024 / d.C;
        if (G < 1) G = 1;
        if (G > d.N) G = d.N;
        g.npg = ceil_div(d.N, G);
        g.G = ceil_div(d.N, g.npg);
        g.rows_per_block = 0;
        g.chunks = g.RP = 1;
    }
    if (d.layout == NSK_NCHW) {
        g.sn = (long)d.C * g.HW;
        g.sc = g.HW;
        g.ss = 1;
    } else {
        g.sn = g.HW * d.C;
        g.sc = 1;
        g.ss = d.C;
    }
    return g;
}

int stream_blocks(long work_items, int per_block = 256)
{
    long b = (work_items + per_block - 1) / per_block;
    const long cap = 256 * 16;  // 16 blocks per CU keep every CU streaming
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

// Thousands of rows of statistics are folded into at most G (what the workspace holds) before the finalize kernel, a block per
// channel, reads them column by column.  That kernel alone takes 0.5-0.9 ns a row while the sums fit an L2 of 4 MB, and
// 1.2-2 ns beyond, since every block then fetches whole cache lines for its four bytes a row; a fold block takes 21 ns a
// row of its share.  So with few blocks (the general path: 1024 / C, at most one an image) folding only pays beyond 4 MB, or
// from 48 blocks on where the rows are very many (us for both, NCHW, folded / not: 32 channels G=32 20 k rows 19 / 36, 50 k 38 /
// 82; 40 channels G=24 15 k 20 / 32; 20 channels G=32 30 k 26 / 42; 8 channels G=48 20 k 15 / 21, 50 k 28 / 46; with four loads
// on their way and 34 ns a row: 40 channels G=24 10 k 20 / 13, 20 channels G=3 10 k 110 / 10, 512 channels G=2 1540 / 77; from
// G=64 on folding never loses above 1024 rows).
bool fold_pays(int stats_rows, int C, const Geom &g)
{
    if (stats_rows <= 1024 || stats_rows <= g.G) return false;
    return g.G >= 64 || (g.G >= 24 && (long)stats_rows * C * 8 > (4L << 20)) || (g.G >= 48 && stats_rows > 16384);
}

dim3 apply_grid(const Geom &g) { return dim3(stream_blocks(g.M, g.RP), g.chunks); }

// f(std::integral_constant<int, VEC>): the access width of the NHWC path as a constant
template <typename T, typename F> void with_vec(const Geom &g, F f)
{
    if constexpr (sizeof(T) == 2) {
        if (g.vec == 8) return f(std::integral_constant<int, 8>{});
    }
    f(std::integral_constant<int, 4>{});
}

// Blocks of the passes over nhwc_fast tensors: rows of sums (never more than the workspace holds) and apply blocks per chunk
int fast_chunk(const nsk_bn_desc_t &d) { return std::min(d.C, d.C > 128 ? kBnChunk : 64); }
int fast_chunks(const nsk_bn_desc_t &d) { return d.C / fast_chunk(d); }
int fast_rows_at_once(const nsk_bn_desc_t &d, int vec) { return kBnThreads / (fast_chunk(d) / vec); }
// Up to 16 MB a tensor (backward 26) the apply blocks finish the sums; larger ones stream better through the many small blocks of the other channel
// counts, which a block of 1024 threads per CU does not replace (both passes of a direction, us, finished in a launch of
// its own / by the apply pass: forward behind a convolution bf16 2 MB 5.5 / 4.9, 13 MB 10.4 / 9.9, 26 MB 13.7 / 14.4, 51 MB 23.4 / 24.9;
// backward with a mask, by_xcd, 64 .. 1024 channels bf16 16 MB 27.4-31.1 / 21.7-22.9, 20 MB 30.2-32.0 / 26.0-27.5, 25 MB 33.6-35.6 / 31.4-34.4, 32 MB 41.0-44.2 /
// 38.5-46.2; fp32 20 MB 27.6-29.7 / 24.8-25.9, 25 MB 31.5-32.9 / 29.6-32.1, 32 MB 38.9-41.1 / 39.0-44.7)
bool apply_finishes(const nsk_bn_desc_t &d, const Geom &g, bool backward) { return g.total * (long)elem_size(d.dtype) <= (backward ? 26L << 20 : 16L << 20); }
int fast_sum_blocks(const nsk_bn_desc_t &d, const Geom &g)
{
    const long passes = (g.M + fast_rows_at_once(d, g.vec) - 1) / fast_rows_at_once(d, g.vec);
    return (int)std::max(1L, std::min<long>({passes, 256 / fast_chunks(d), (long)g.G}));
}
// Backward with a mask that was handed over, from 150 MB a tensor on (fp32 with one or two chunks: 30 MB): blocks of 256 threads, two
// a CU, as the other channel counts (64 channels, both passes, us, blocks of 1024 / of 256 threads: fp32 51 MB 48.2 / 47.1, 205 MB
// 172 / 167, 411 MB 372 / 341; bf16 205 MB 174 / 170, but 26 MB 29.4 / 30.8; fp32 103 MB of 1024 channels 87 / 93)
bool many_small_sums(const nsk_bn_desc_t &d, const Geom &g, bool mask_in)
{
    return mask_in && g.total * (long)elem_size(d.dtype) >= (d.dtype == NSK_F32 && d.C <= 128 ? 30L << 20 : 150L << 20);
}
dim3 fast_apply_grid(const nsk_bn_desc_t &d, const Geom &g)
{
    const long passes = (g.M + fast_rows_at_once(d, g.vec) - 1) / fast_rows_at_once(d, g.vec);
    return dim3((unsigned)std::max(1L, std::min<long>(passes, 256 / fast_chunks(d))), fast_chunks(d));
}
// Forward, its own statistics: the sums in chunks pay where 512 blocks over whole rows would leave many of them to the launch between, or
// the tensor is large; below, two launches of 1024 threads a block with their sums in LDS take longer than the three of the other
// channel counts (us, those / these: bf16 64 channels 0.4, 1.6, 4, 11 MB 8.4 / 9.2, 9.3 / 10.2, 10.1 / 10.9, 14.9 / 14.7; 256 channels 0.4, 4, 8, 12
// MB 8.4 / 10.3, 10.6 / 12.1, 14.4 / 14.7, 17.1 / 16.4; 512 channels 3, 6 MB 11.7 / 12.1, 15.4 / 13.8; 1024 channels 0.4, 1.5 MB 9.8 / 9.9, 11.7 / 10.7;
// fp32 64 channels 4, 8, 11 MB 8.6 / 9.9, 10.9 / 11.8, 12.7 / 13.1; 256 channels 8, 11 MB 12.5 / 12.6, 14.9 / 13.6)
// At 16 MB sharp, a common size, they are slower than at 15 and 17 MB (64 channels bf16 16.6 and 17.7 us), the cause not known: up to 128
// channels the three launches again (64 channels, those / sums in chunks with a launch between / finished by the apply pass: bf16 16.7 / 18.2 / 19.1, fp32 14.4 / 15.8 /
// 16.1; 256 channels 19.4 / 19.0 / 20.5, 17.1 / 15.9 / 16.2).
bool own_sums_fast(const nsk_bn_desc_t &d, const Geom &g)
{
    const long bytes = g.total * (long)elem_size(d.dtype);
    return bytes >= (d.C >= 1024 ? 0L : d.C >= 512 ? 4L << 20 : 10L << 20) && (bytes != 16L << 20 || d.C > 128);
}
// Statistics of a convolution: every apply block reads the sums of its chunk, so they must be few; up to 100 KB a chunk that beats the
// launch between (0.78-1.04 of its time), 200 KB up to 32 channels, 220 KB from 512, 512 KB from 1024 channels on, where that launch reads
// column by column for long (us, launch between / apply pass: bf16 64 channels, 1.6 MB, 64, 196, 256, 784 rows 4.9 / 4.3, 5.3 / 5.1, 5.5 / 5.1, 6.0 /
// 7.3; 256 channels, 3 MB, 64, 256, 784 rows 5.9 / 5.6, 6.1 / 6.7, 7.3 / 8.6; 1024 channels, 6 MB, 256 rows 9.2 / 9.0; 16 channels, 784 rows 5.4 /
// 5.2; with the convolution in front, 512 channels, 12 MB, 196 rows 29.0 / 27.1, 256 channels, 3 MB, 196 rows 13.4 / 13.9)
bool rows_fit_apply(int rows, const nsk_bn_desc_t &d)
{
    const long kb = d.C >= 1024 ? 512 : d.C >= 512 ? 220 : d.C > 32 ? 100 : 200;
    return (long)rows * fast_chunk(d) * 8 <= kb << 10;
}
// Above 1024 rows (512 channels and more: 512) they are folded first, by enough blocks, if the apply pass cannot read them (launch between / fold and apply pass, us: 64 channels, 3 MB, 784, 1568 rows 6.4 / 7.9, 8.0 / 7.2; 512 channels, 6 MB, 784 rows
// 10.5 / 10.4; 12 MB, 1024 rows 15.0 / 12.3)
bool fold_first(int stats_rows, const nsk_bn_desc_t &d, const Geom &g)
{
    return g.G >= 16 && stats_rows > (d.C >= 512 ? 512 : 1024) && !rows_fit_apply(stats_rows, d);
}
// Sums and apply pass by eighths of the rows (walk_rows), where there are sums and the apply pass finishes them: from 4.1 MB on, where the apply pass
// begins to miss what it needs in its own L2 (backward, 64 .. 1024 channels, us, rows in one piece / by eighths: bf16 4.0 MB 10.4-11.6 / 10.5-11.6, 4.2 MB
// 14.0-14.9 / 10.8-12.7, 6 MB 15.4-16.3 / 11.6-12.4, 8 MB 16.2-17.9 / 11.9-12.9, 12 MB 20.4-21.4 / 14.3-15.6, 15.9 MB 27.6-30.2 / 21.5-23.2; fp32 4.0 MB 9.2-10.4 /
// 9.2-10.5, 4.6 MB 12.5-13.3 / 10.1-10.9, 12 MB 18.2-19.3 / 12.8-14.2; forward with its own statistics, 12 MB 14.3-17.6 / 13.7-17.1, 15.9 MB 17.0-20.9 /
// 15.3-18.9; behind a convolution, whose own blocks wrote x, no difference)
bool by_xcd(const nsk_bn_desc_t &d, const Geom &g, bool finish)
{
    return finish && g.total * (long)elem_size(d.dtype) >= (4200L << 10) && fast_sum_blocks(d, g) % 8 == 0 && fast_apply_grid(d, g).x % 8 == 0;
}
template <typename T, int MODE, int THREADS>
void launch_sums_fast(const nsk_bn_desc_t &d, const Geom &g, int G, bool xcd, const T *x, const T *out, const T *dout, const float *mean, const float *invstd,
                      float *p0, float *p1, unsigned char *mask, const unsigned char *mask_in, const float *act, float *shift, hipStream_t stream)
{
    constexpr int VEC = 16 / (int)sizeof(T);
    const size_t lds = (size_t)THREADS * VEC * 2 * sizeof(float);
    auto go = [&](auto X) {
        hipLaunchKernelGGL((bn_sums_fast<T, VEC, MODE, THREADS, X.value>), dim3(G, fast_chunks(d)), dim3(THREADS), lds, stream, x, out, dout, mean,
                           invstd, d.relu, g.M, d.C, (g.M + G - 1) / G, p0, p1, mask, mask_in, act, shift);
    };
    if constexpr (THREADS == kBnThreads) {
        if (xcd) return go(std::true_type{});
    }
    go(std::false_type{});
}

template <typename T>
int bn_fwd_fast(const nsk_bn_desc_t &d, const Geom &g, bool xcd, const T *x, const T *res, T *out, unsigned char *relu_mask, const BnFwdFinish &f, hipStream_t stream)
{
    constexpr int VEC = 16 / (int)sizeof(T);
#define NSK_APPLY(R, L) \
        hipLaunchKernelGGL((bn_apply_fast<T, VEC, R, L, X.value>), fast_apply_grid(d, g), dim3(kBnThreads), 0, stream, x, res, out, g.M, d.C, relu_mask, f)
    auto go = [&](auto X) {
        if (res) {
            if (d.relu) NSK_APPLY(true, true); else NSK_APPLY(true, false);
        } else {
            if (d.relu) NSK_APPLY(false, true); else NSK_APPLY(false, false);
        }
    };
    if (xcd) go(std::true_type{}); else go(std::false_type{});
#undef NSK_APPLY
    return check_launch();
}

template <typename T>
int bn_bwd_fast(const nsk_bn_desc_t &d, const Geom &g, bool xcd, const T *x, const T *dout, T *dx, T *dres, const unsigned char *mask, const BnBwdFinish &f, hipStream_t stream)
{
    constexpr int VEC = 16 / (int)sizeof(T);
#define NSK_BAPPLY(R, L) \
        hipLaunchKernelGGL((bn_bwd_apply_fast<T, VEC, R, L, X.value>), fast_apply_grid(d, g), dim3(kBnThreads), 0, stream, x, dout, dx, dres, g.M, d.C, mask, f)
    auto go = [&](auto X) {
        if (dres) {
            if (d.relu) NSK_BAPPLY(true, true); else NSK_BAPPLY(true, false);
        } else {
            if (d.relu) NSK_BAPPLY(false, true); else NSK_BAPPLY(false, false);
        }
    };
    if (xcd) go(std::true_type{}); else go(std::false_type{});
#undef NSK_BAPPLY
    return check_launch();
}

template <typename T>
int bn_fwd_typed(const nsk_bn_desc_t &d, const T *x, const T *res, const float *gamma, const float *beta, T *out,
                 float *save_mean, float *save_invstd, float *running_mean, float *running_var, float *ws,
                 unsigned char *relu_mask, const float *stats, int stats_rows, hipStream_t stream)
{
    const Geom g = geometry(d, false);
    const bool fast = nhwc_fast(d) && (stats || own_sums_fast(d, g));
    // (with its own statistics at 16 MB sharp no longer: own_sums_fast)
    bool finish = fast && apply_finishes(d, g, false) && (stats || g.total * (long)sizeof(T) < (16L << 20));
    float *p0 = ws, *p1 = ws + (long)g.G * d.C, *scale = p1 + (long)g.G * d.C, *bias = scale + d.C;
    const bool xcd = !stats && by_xcd(d, g, finish);
    const float *q0 = p0, *q1 = p1;
    int rows = fast ? fast_sum_blocks(d, g) : g.G;
    if (stats) {
        // partial sums of x and x^2 left by the producer of x ([2][stats_rows][C], not shifted): no reduction pass.
        // A producer with small tiles leaves tens of thousands of rows: those are first folded into at most G rows
        // (the finalize kernel has one wavefront per channel).
        q0 = stats;
        q1 = stats + (long)stats_rows * d.C;
        rows = stats_rows;
        if (finish ? fold_first(stats_rows, d, g) : fold_pays(stats_rows, d.C, g)) {
            // few rows for the launch behind, but 64 of them at most for a block here (64 MB of 256 channels, 3136 rows into 512 / 64 39.7 / 31.2 us;
            // 24 MB of 16 channels, 16384 rows 16.1 / 20.1)
            const int run = ceil_div(stats_rows, fast ? std::min(g.G, std::max(64, ceil_div(stats_rows, 64))) : g.G);
            rows = ceil_div(stats_rows, run);
            hipLaunchKernelGGL(bn_stats_fold, dim3(rows, ceil_div(2 * d.C, 256)), dim3(256), 0, stream, stats, stats_rows, d.C, run, p0, rows);
            q0 = p0;
            q1 = p0 + (long)rows * d.C;
        }
        finish = finish && rows_fit_apply(rows, d);
    } else if (fast) {
        launch_sums_fast<T, 0, kBnThreads>(d, g, rows, xcd, x, nullptr, nullptr, nullptr, nullptr, p0, p1, nullptr, nullptr, nullptr, scale, stream);
    } else if (g.vec) {
        with_vec<T>(g, [&](auto V) {
            hipLaunchKernelGGL((bn_reduce_nhwc<T, V.value, 0>), dim3(g.G, g.chunks), dim3(256), 0, stream, x, (const T *)nullptr,
                               (const T *)nullptr, (const float *)nullptr, (const float *)nullptr, 0, g.M, d.C,
                               g.rows_per_block, p0, p1, 0);
        });
    } else {
        hipLaunchKernelGGL((bn_reduce_generic<T, 0>), dim3(d.C, g.G), dim3(256), 0, stream, x, (const T *)nullptr,
                           (const T *)nullptr, (const float *)nullptr, (const float *)nullptr, 0, d.N, g.HW, g.sn,
                           g.sc, g.ss, g.npg, d.C, p0, p1);
    }
    const BnFwdFinish f{q0, q1, gamma, beta, stats ? nullptr : scale, save_mean, save_invstd, running_mean, running_var, (double)g.M, d.eps, d.momentum, rows};
    if (finish) return bn_fwd_fast<T>(d, g, xcd, x, res, out, relu_mask, f, stream);
    hipLaunchKernelGGL((bn_fwd_finalize<T>), dim3(d.C), dim3(256), 0, stream, q0, q1, rows, d.C, (double)g.M, stats ? (const T *)nullptr : x,
                       stats ? 0L : g.sc, gamma, beta, d.eps, d.momentum, save_mean, save_invstd, running_mean, running_var, scale, bias);
    if (g.vec) {
        const long nvec = g.total / g.vec;
        const dim3 grid = apply_grid(g);
#define NSK_APPLY(R, L) \
    hipLaunchKernelGGL((bn_apply_nhwc<T, V.value, R, L>), grid, dim3(256), 0, stream, x, res, out, scale, bias, nvec, d.C, relu_mask)
        with_vec<T>(g, [&](auto V) {
            if (res) {
                if (d.relu) NSK_APPLY(true, true); else NSK_APPLY(true, false);
            } else {
                if (d.relu) NSK_APPLY(false, true); else NSK_APPLY(false, false);
            }
        });
#undef NSK_APPLY
    } else {
        const dim3 grid(stream_blocks(g.total));
        if (d.layout == NSK_NCHW)
            hipLaunchKernelGGL((bn_apply_generic<T, true>), grid, dim3(256), 0, stream, x, res, out, scale, bias,
                               g.total, d.C, g.HW, d.relu);
        else
            hipLaunchKernelGGL((bn_apply_generic<T, false>), grid, dim3(256), 0, stream, x, res, out, scale, bias,
                               g.total, d.C, g.HW, d.relu);
    }
    return check_launch();
}

template <typename T>
int bn_bwd_typed(const nsk_bn_desc_t &d, const T *x, const T *out, const T *dout, const float *gamma,
                 const float *mean, const float *invstd, T *dx, T *dres, float *dgamma, float *dbeta, float *ws,
                 const unsigned char *mask_in, hipStream_t stream, const float *act = nullptr)
{
    const Geom g = geometry(d, true);
    const bool masked = nhwc_fast(d);   // the ReLU mask goes from pass to pass; else both read out
    if (act && !(masked && d.relu)) return NSK_ERR_UNSUPPORTED;
    float *p0 = ws, *p1 = ws + (long)g.G * d.C, *coef = p1 + (long)g.G * d.C;
    // the ReLU mask bytes follow the float part of the workspace (see bn_mask_bytes)
    unsigned char *mask = (unsigned char *)ws + align_up((2 * (size_t)bn_partial_blocks(d) * d.C + 4 * (size_t)d.C) * sizeof(float));
    const unsigned char *kept = mask_in ? mask_in : mask;
    const bool finish = masked && apply_finishes(d, g, true), xcd = by_xcd(d, g, finish);
    const bool many = !finish && many_small_sums(d, g, mask_in != nullptr);
    const int rows = masked && !many ? fast_sum_blocks(d, g) : many ? std::min(g.G, 512 / fast_chunks(d)) : g.G;
    if (masked && act) {
        launch_sums_fast<T, 2, kBnThreads>(d, g, rows, xcd, x, out, dout, mean, invstd, p0, p1, mask, nullptr, act, nullptr, stream);
    } else if (masked && many) {
        launch_sums_fast<T, 1, 256>(d, g, rows, false, x, out, dout, mean, invstd, p0, p1, mask, mask_in, nullptr, nullptr, stream);
    } else if (masked) {
        launch_sums_fast<T, 1, kBnThreads>(d, g, rows, xcd, x, out, dout, mean, invstd, p0, p1, mask, mask_in, nullptr, nullptr, stream);
    } else if (g.vec) {
        with_vec<T>(g, [&](auto V) {
            hipLaunchKernelGGL((bn_reduce_nhwc<T, V.value, 1>), dim3(g.G, g.chunks), dim3(256), 0, stream, x, out, dout, mean, invstd,
                               d.relu, g.M, d.C, g.rows_per_block, p0, p1, 0);
        });
    } else {
        hipLaunchKernelGGL((bn_reduce_generic<T, 1>), dim3(d.C, g.G), dim3(256), 0, stream, x, out, dout, mean,
                           invstd, d.relu, d.N, g.HW, g.sn, g.sc, g.ss, g.npg, d.C, p0, p1);
    }
    const BnBwdFinish f{p0, p1, gamma, mean, invstd, dgamma, dbeta, (double)g.M, rows};
    if (finish) return bn_bwd_fast<T>(d, g, xcd, x, dout, dx, dres, kept, f, stream);
    hipLaunchKernelGGL(bn_bwd_finalize, dim3(d.C), dim3(256), 0, stream, p0, p1, rows, d.C,
                       (double)g.M, gamma, invstd, dgamma, dbeta, coef);
    if (g.vec) {
        const long nvec = g.total / g.vec;
        const dim3 grid = apply_grid(g);
#define NSK_BAPPLY(R, L)                                                                                       \
    hipLaunchKernelGGL((bn_bwd_apply_nhwc<T, V.value, R, L>), grid, dim3(256), 0, stream, x, out, dout, dx, dres, mean, \
                       invstd, coef, nvec, d.C, kept)
        with_vec<T>(g, [&](auto V) {
            if (dres) {
                if (!d.relu) NSK_BAPPLY(true, 0); else if (masked) NSK_BAPPLY(true, 1); else NSK_BAPPLY(true, 2);
            } else {
                if (!d.relu) NSK_BAPPLY(false, 0); else if (masked) NSK_BAPPLY(false, 1); else NSK_BAPPLY(false, 2);
            }
        });
#undef NSK_BAPPLY
    } else {
        const dim3 grid(stream_blocks(g.total));
        if (d.layout == NSK_NCHW)
            hipLaunchKernelGGL((bn_bwd_apply_generic<T, true>), grid, dim3(256), 0, stream, x, out, dout, dx, dres,
                               mean, invstd, coef, g.total, d.C, g.HW, d.relu);
        else
            hipLaunchKernelGGL((bn_bwd_apply_generic<T, false>), grid, dim3(256), 0, stream, x, out, dout, dx, dres,
                               mean, invstd, coef, g.total, d.C, g.HW, d.relu);
    }
    return check_launch();
}

}  // namespace

// Bytes of ReLU mask the backward pass keeps between its two kernels (one byte per 16-byte vector), 0 if unused.
size_t bn_mask_bytes(const nsk_bn_desc_t &d)
{
    if (!d.relu || !nhwc_fast(d)) return 0;
    const size_t vec = d.dtype == NSK_BF16 ? 8 : 4;
    return (size_t)d.N * d.H * d.W * d.C / vec;
}

int bn_partial_blocks(const nsk_bn_desc_t &d)
{
    const int f = geometry(d, false).G, b = geometry(d, true).G;
    return f > b ? f : b;
}

int launch_bn_fwd(const nsk_bn_desc_t &d, const void *x, const void *residual, const float *gamma,
                  const float *beta, void *out, float *save_mean, float *save_invstd, float *running_mean,
                  float *running_var, void *ws, unsigned char *relu_mask, const float *stats, int stats_rows,
                  hipStream_t stream)
{
    if (d.dtype == NSK_BF16)
        return bn_fwd_typed<bf16_t>(d, (const bf16_t *)x, (const bf16_t *)residual, gamma, beta, (bf16_t *)out,
                                    save_mean, save_invstd, running_mean, running_var, (float *)ws, relu_mask, stats,
                                    stats_rows, stream);
    return bn_fwd_typed<float>(d, (const float *)x, (const float *)residual, gamma, beta, (float *)out, save_mean,
                               save_invstd, running_mean, running_var, (float *)ws, relu_mask, stats, stats_rows, stream);
}

// Partial sums of x and x^2 per channel, [2][rows][C] floats (bn_stats_rows(d) of them are best), not shifted: what the convolution kernels
// with a fused statistics epilogue write, produced here by a reduction pass for the shapes they do not cover.
int bn_stats_rows(const nsk_bn_desc_t &d) { return geometry(d, false).G; }

int launch_bn_stats(const nsk_bn_desc_t &d, const void *x, float *stats, int rows, hipStream_t stream)
{
    Geom g = geometry(d, false);
    if (rows != g.G) {      // blocks past the end of the tensor leave zeros
        g.G = rows;
        g.rows_per_block = (g.M + rows - 1) / rows;
        g.npg = ceil_div(d.N, rows);
    }
    float *p0 = stats, *p1 = stats + (long)g.G * d.C;
#define NSK_STATS(T)                                                                                                   \
    if (g.vec)                                                                                                         \
        with_vec<T>(g, [&](auto V) {                                                                                   \
            hipLaunchKernelGGL((bn_reduce_nhwc<T, V.value, 0>), dim3(g.G, g.chunks), dim3(256), 0, stream, (const T *)x, \
                               (const T *)nullptr, (const T *)nullptr, (const float *)nullptr, (const float *)nullptr, \
                               0, g.M, d.C, g.rows_per_block, p0, p1, 1);                                              \
        });                                                                                                            \
    else                                                                                                               \
        hipLaunchKernelGGL((bn_reduce_generic<T, 0>), dim3(d.C, g.G), dim3(256), 0, stream, (const T *)x,              \
                           (const T *)nullptr, (const T *)nullptr, (const float *)nullptr, (const float *)nullptr, 0,  \
                           d.N, g.HW, g.sn, g.sc, g.ss, g.npg, d.C, p0, p1, 1)
    if (d.dtype == NSK_BF16) {
        NSK_STATS(bf16_t);
    } else {
        NSK_STATS(float);
    }
#undef NSK_STATS
    return check_launch();
}

int launch_bn_bwd(const nsk_bn_desc_t &d, const void *x, const void *out, const void *dout, const float *gamma,
                  const float *save_mean, const float *save_invstd, void *dx, void *dres, float *dgamma,
                  float *dbeta, void *ws, const unsigned char *relu_mask, hipStream_t stream, const float *act)
{
    if (d.dtype == NSK_BF16)
        return bn_bwd_typed<bf16_t>(d, (const bf16_t *)x, (const bf16_t *)out, (const bf16_t *)dout, gamma,
                                    save_mean, save_invstd, (bf16_t *)dx, (bf16_t *)dres, dgamma, dbeta,
                                    (float *)ws, relu_mask, stream, act);
    return bn_bwd_typed<float>(d, (const float *)x, (const float *)out, (const float *)dout, gamma, save_mean,
                               save_invstd, (float *)dx, (float *)dres, dgamma, dbeta, (float *)ws, relu_mask, stream, act);
}

// True if the fused-activation calls take this tensor: NHWC with a channel count the vector kernels handle.
bool bn_act_supported(const nsk_bn_desc_t &d) { return nhwc_fast(d); }

// Batch statistics and the coefficients of out = scale*x + shift (scale = gamma*invstd, shift = beta - mean*scale) from
// partial sums of x and x^2 ([2][stats_rows][C], not shifted), without the apply pass: coeffs = [2][C] floats.
int launch_bn_coeffs(const nsk_bn_desc_t &d, const float *gamma, const float *beta, const float *stats, int stats_rows,
                     float *save_mean, float *save_invstd, float *running_mean, float *running_var, float *coeffs,
                     void *ws, hipStream_t stream)
{
    const Geom g = geometry(d, false);
    float *p0 = (float *)ws;
    const float *q0 = stats, *q1 = stats + (long)stats_rows * d.C;
    int rows = stats_rows;
    if (fold_pays(stats_rows, d.C, g)) {
        const int run = ceil_div(stats_rows, g.G), r2 = ceil_div(stats_rows, run);
        hipLaunchKernelGGL(bn_stats_fold, dim3(r2), dim3(256), 0, stream, stats, stats_rows, d.C, run, p0, r2);
        q0 = p0;
        q1 = p0 + (long)r2 * d.C;
        rows = r2;
    }
    if (d.dtype == NSK_BF16)
        hipLaunchKernelGGL((bn_fwd_finalize<bf16_t>), dim3(d.C), dim3(256), 0, stream, q0, q1, rows, d.C, (double)g.M,
                           (const bf16_t *)nullptr, 0L, gamma, beta, d.eps, d.momentum, save_mean, save_invstd,
                           running_mean, running_var, coeffs, coeffs + d.C);
    else
        hipLaunchKernelGGL((bn_fwd_finalize<float>), dim3(d.C), dim3(256), 0, stream, q0, q1, rows, d.C, (double)g.M,
                           (const float *)nullptr, 0L, gamma, beta, d.eps, d.momentum, save_mean, save_invstd,
                           running_mean, running_var, coeffs, coeffs + d.C);
    return check_launch();
}

// out = relu(scale*x + shift) with the coefficients of launch_bn_coeffs: the apply pass on its own, for consumers
// whose kernel has no fused operand load.
int launch_bn_act(const nsk_bn_desc_t &d, const void *x, const float *coeffs, void *out, hipStream_t stream)
{
    const Geom g = geometry(d, false);
    if (!nhwc_fast(d)) return NSK_ERR_UNSUPPORTED;
    const long nvec = g.total / g.vec;
    if (d.dtype == NSK_BF16)
        hipLaunchKernelGGL((bn_apply_nhwc<bf16_t, 8, false, true>), apply_grid(g), dim3(256), 0, stream, (const bf16_t *)x,
                           (const bf16_t *)nullptr, (bf16_t *)out, coeffs, coeffs + d.C, nvec, d.C, (unsigned char *)nullptr);
    else
        hipLaunchKernelGGL((bn_apply_nhwc<float, 4, false, true>), apply_grid(g), dim3(256), 0, stream, (const float *)x,
                           (const float *)nullptr, (float *)out, coeffs, coeffs + d.C, nvec, d.C, (unsigned char *)nullptr);
    return check_launch();
}

}  // namespace nsk
