// Internal declarations shared by the translation units of libnsk (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "nsk.h"

namespace nsk {

typedef __bf16 bf16_t;
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMaxTaps = 64;    // R*S of one launch (a 7x7 filter has 49)
constexpr int kMaxBnChannels = 4096;

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline size_t elem_size(int dtype) { return dtype == NSK_BF16 ? 2 : 4; }

// Compile-time loop: f(std::integral_constant<int, B>), ..., f(std::integral_constant<int, E - 1>).  For loop bodies
// whose index must be a constant expression (register arrays, per-iteration schedules chosen with `if constexpr`).
template <int B, int E, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Block-wide barrier that orders LDS traffic only.  __syncthreads() also drains the wavefront's global loads
// (its fence covers global memory), which would end every register prefetch at each barrier; kernels whose
// wavefronts exchange data through LDS alone use this one and keep their loads in flight across it.
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Until at most N of the wavefront's direct loads (memory to LDS) are on their way and all its LDS reads have arrived: a barrier
// behind it then also says that nobody reads the stage before any more.
template <int N> __device__ inline void wait_vm()
{
    static_assert(N >= 0 && N < 64, "six-bit counter");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

// n / d for 0 <= n < 2^31 as (n * mul) >> sh with mul = ceil(2^(31+s) / d), s = ceil(log2 d), sh = 31 + s
struct Div {
    unsigned mul;
    int sh;
};
inline Div make_div(int d)
{
    int s = 0;
    while ((1LL << s) < d) ++s;
    Div r;
    r.mul = (unsigned)(((1ULL << (31 + s)) + (unsigned)d - 1) / (unsigned)d);
    r.sh = 31 + s;
    return r;
}
__device__ inline int divide(int n, const Div &d) { return (int)(((unsigned long long)(unsigned)n * d.mul) >> d.sh); }

// fp32 products on the bf16 matrix unit.  x = h + m + l exactly, three bf16 pieces (h and m to nearest, l what is left: 8 + 8 + 8 bits),
// and x*y = hh' + (hm' + mh') + (mm' + hl' + lh') + terms below 2^-24 of it: six bf16
// products of 16 indices in place of eight fp32 ones of 2, in 192 clocks instead of 512, and with fewer roundings of the sums.  What is left out
// leaves a sum of one product, which the fp32 unit rounds once, 0.60e-7 of it at most and 2.53e-8 rms, off by 1.0e-7 at most (2^-23 is the bound) and
// 2.58e-8 rms; sums of two are off by 2.6e-8 rms (fp32 unit 3.1e-8), of 16 by 3.1e-8 (7.4e-8).  (m cut instead of rounded: 1.5e-7 and 2.9e-8 for one.  With
// ml' and lm', eight products, one is rounded as on the fp32 unit, but units take 8-12% longer and small ones longer than on the fp32 unit: 64 -> 64 3x3 at
// 32x32, N=16, 22.3 us, here 17.3, there 15.7.)  What the vector unit spends on the pieces, 13 instructions for two values, bounds it: a wavefront
// should multiply each piece it makes several times.
// Both operands are multiplied by 2^24 first and the sums by 2^-48 at the end: the last bit of the smallest float, 2^-149, then is a whole bf16,
// 2^-125, and every finite operand has exact pieces (unscaled, the last piece of |x| < 2^-110 leaves the range of bf16, and gradients that
// vanish over a long sequence, or decayed filters, get there).  A value that is not finite or too large for that (2^104, products 2^80) makes sums
// that are not finite: a kernel that sees such (finite_sums) makes them again on the fp32 unit.
struct Pieces {
    bf16x8 h, m, l;
};
constexpr float kPieceScale = 16777216.f, kSumScale = kPieceScale * kPieceScale;
__device__ __forceinline__ Pieces split3(const float (&x)[8])
{
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
    struct Quad {
        unsigned q[4];
    } h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i] * kPieceScale, b = x[2 * i + 1] * kPieceScale;
        bf16x2 p;
        p[0] = (bf16_t)a;
        p[1] = (bf16_t)b;
        h.q[i] = __builtin_bit_cast(unsigned, p);
        asm("" : "+v"(h.q[i]));     // (else the compiler rounds a second time instead of shifting)
        float ra = a - __builtin_bit_cast(float, h.q[i] << 16), rb = b - __builtin_bit_cast(float, h.q[i] & 0xffff0000u);
        p[0] = (bf16_t)ra;
        p[1] = (bf16_t)rb;
        m.q[i] = __builtin_bit_cast(unsigned, p);
        asm("" : "+v"(m.q[i]));
        ra -= __builtin_bit_cast(float, m.q[i] << 16);
        rb -= __builtin_bit_cast(float, m.q[i] & 0xffff0000u);
        l.q[i] = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, rb), __builtin_bit_cast(unsigned, ra), 0x07060302u);
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
// hi + lo += sum over 16 indices of x[i] * y[j], x the matrix unit's first operand; sums at [i][j], or [j][i] where SECOND_ROWS.  Where lo is
// not hi, the large products have accumulators of their own: a sum is then rounded at its full size once in 16 indices, not six times.
template <bool SECOND_ROWS, int FX, int FY, int R, int C>
__device__ __forceinline__ void multiply_pieces(const Pieces (&x)[FX], const Pieces (&y)[FY], f32x16 (&hi)[R][C], f32x16 (&lo)[R][C])
{
    static_assert(R == (SECOND_ROWS ? FY : FX) && C == (SECOND_ROWS ? FX : FY), "one sum a pair");
#define NSK_PRODUCT(P, Q, S) S[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i].P, y[j].Q, S[r][c], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const int c = r & 1 ? C - 1 - k : k, i = SECOND_ROWS ? c : r, j = SECOND_ROWS ? r : c;
            NSK_PRODUCT(h, l, lo)
            NSK_PRODUCT(h, h, hi)
            NSK_PRODUCT(l, h, lo)
            NSK_PRODUCT(m, m, lo)
            NSK_PRODUCT(h, m, lo)
            NSK_PRODUCT(m, h, lo)
        }
#undef NSK_PRODUCT
}
// This lane's sums are all finite.
template <int FM, int FN> __device__ __forceinline__ bool finite_sums(const f32x16 (&acc)[FM][FN])
{
    // largest magnitude by bits: infinities and NaN above all numbers
    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const unsigned u = __builtin_bit_cast(unsigned, acc[i][j][v]) & 0x7fffffffu;
                top = u > top ? u : top;
            }
    return top < 0x7f800000u;
}

// The value of lane ^ O: O = 2, 4, 8 within a row of 16 lanes, on the vector unit.
template <int O> __device__ __forceinline__ float lane_xor(float v)
{
    auto moved = [](float x, auto ctl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctl)::value, 0xf, 0xf, true));
    };
    static_assert(O == 2 || O == 4 || O == 8, "within a row");
    if constexpr (O == 2) return moved(v, std::integral_constant<int, 0x4e>{});      // quad_perm 2,3,0,1
    else if constexpr (O == 8) return moved(v, std::integral_constant<int, 0x128>{});     // row_ror 8
    else return moved(moved(v, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1b>{});     // row_half_mirror, quad_perm 3,2,1,0
}
// Sums of N values over the lanes with the same lane % CPP.  Each step halves what a lane still carries: it hands the half that the other
// lane goes on with over for the half that it goes on with itself (N/2 + N/4 + ... exchanges, where adding every value across all lanes
// takes N a step, each an LDS operation; those of lanes 32 and 16 apart are swaps of registers).  Neighbours first: the same sums bit by bit
// as v += v of lane ^ CPP, then of lane ^ 2 * CPP, up to lane ^ 32.  Afterwards lane l holds value l / CPP % (64 / CPP) of its lanes in v[0], that plus 64 / CPP in
// v[1], and so on (N < 64 / CPP: value l / CPP % N).
template <int CPP, int N, int O = CPP, int LEFT = N> __device__ __forceinline__ void fold_lanes(float (&v)[N])
{
    if constexpr (O < 64) {
        constexpr int H = LEFT / 2;
        if constexpr (O >= 16) {
#pragma unroll
            for (int i = 0; i < (H > 0 ? H : 1); ++i) {
                const unsigned a = __builtin_bit_cast(unsigned, v[H > 0 ? 2 * i : 0]), b = __builtin_bit_cast(unsigned, v[H > 0 ? 2 * i + 1 : 0]);
                const auto r = O == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false) : __builtin_amdgcn_permlane16_swap(a, b, false, false);
                v[i] = __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
            }
        } else if constexpr (LEFT == 1) {
            v[0] += lane_xor<O>(v[0]);
        } else {
            const bool upper = (threadIdx.x & O) != 0;
#pragma unroll
            for (int i = 0; i < H; ++i) v[i] = (upper ? v[2 * i + 1] : v[2 * i]) + lane_xor<O>(upper ? v[2 * i] : v[2 * i + 1]);
        }
        fold_lanes<CPP, N, O * 2, (H > 0 ? H : 1)>(v);
    }
}

// Statistics of a block's or a wavefront's stores: lane l has added up the 8 channels (l % CPP) * 8 .. + 7 of its rows.  r: a row of partial
// sums from the first of those channels on, its squares `squares` floats further.
template <int CPP> __device__ __forceinline__ void store_folded(const float (&sum)[8], const float (&sq)[8], float *r, size_t squares)
{
    constexpr int LANES = CPP < 4 ? 16 : 64 / CPP, PER = 16 / LANES;      // values a lane ends up with
    const int lane = threadIdx.x & 63;
    float v[16];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = sum[e];
        v[8 + e] = sq[e];
    }
    fold_lanes<CPP>(v);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int value = lane / CPP % LANES + i * LANES;
        r[(value >= 8 ? squares : 0) + lane % CPP * 8 + value % 8] = v[i];
    }
}

// Test and A/B switches: environment variables NSK_*, read ONCE (first use, or nsk_test_hooks_reload()) and never on
// the launch path.  Each one only narrows or widens the choice among kernels that all compute the same result.
struct TestHooks {
    bool no_pw, no_halo, no_fs, no_halo_wide, halo_wide_always, halo64_always, halo_single, no_stem, no_stem_halo,
        no_tiny, no_depthwise, no_grouped8, no_pad, depthwise_no_rows, depthwise_no_cols, pool_general, reduce4,
        wh_no_split, gru_far;
    long long pw_min_rows, wh_min_rows;   // -1: not set
    int igemm_tile, gru_split;                              // 0: not set
    int gru_polls;                                          // -1: not set
};
const TestHooks &hooks();

void set_last_hip_error(hipError_t e);
// Returns NSK_OK or records the error and returns NSK_ERR_HIP.
inline int check_launch()
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return NSK_ERR_HIP;
    }
    return NSK_OK;
}

// Allows a kernel `bytes` of dynamic LDS on the current device: once per device, whose own copy of the function it belongs to.
inline int allow_lds(const void *kernel, size_t bytes, std::atomic<unsigned long long> &done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    const unsigned long long bit = dev < 64 ? 1ull << dev : 0;
    if (e == hipSuccess && (done.load(std::memory_order_relaxed) & bit)) return NSK_OK;
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return NSK_ERR_HIP;
    }
    done.fetch_or(bit, std::memory_order_relaxed);
    return NSK_OK;
}
template <auto KERNEL> struct Kernel {
    static constexpr auto value = KERNEL;
};
template <auto KERNEL> inline int allow_lds(size_t bytes)
{
    static std::atomic<unsigned long long> done{0};
    return allow_lds((const void *)KERNEL, bytes, done);
}

// Compute units of the current device.
inline int compute_units(int *n)
{
    static std::atomic<int> known[64];       // of each device, once asked for
    int dev = 0, c = 0;
    hipError_t e = hipGetDevice(&dev);
    const bool kept = e == hipSuccess && dev >= 0 && dev < 64;
    if (kept) c = known[dev].load(std::memory_order_relaxed);
    if (e == hipSuccess && c == 0) e = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return NSK_ERR_HIP;
    }
    if (kept) known[dev].store(c, std::memory_order_relaxed);
    *n = c > 0 ? c : 256;
    return NSK_OK;
}

// Validated geometry of one convolution descriptor.
struct ConvGeo {
    int N, C, H, W, K, R, S, sh, sw, ph, pw, dh, dw, P, Q;
    int dtype, layout;
    size_t es;
    size_t x_elems, y_elems, w_elems;
};

// ------------------------------------------------------------------ implicit GEMM (fwd, dgrad)
// One launch computes, for every GEMM row m = (img, i, j) with i < Mi, j < Mj and every
// column n < Ngemm:
//   acc[m][n] = sum over taps t and channels c of
//               src[img][i*mult_h + add_h + off_h[t]][j*mult_w + add_w + off_w[t]][c] * wpk[n][t][c]
// (source positions outside [0,Hs) x [0,Ws) count as zero) and stores it, converted to the
// element type, at out[img][i*osh + oa][j*osw + ob][n], adding the old value if `accumulate`.
struct IgemmArgs {
    const void *src;  // NHWC [Nimg][Hs][Ws][Cs]
    const void *wpk;  // [Ngemm][ntaps][Cs]
    void *out;        // NHWC [Nimg][Ho][Wo][Co]
    int Nimg, Hs, Ws, Cs;
    int Mi, Mj, M;
    int mult_h, add_h, mult_w, add_w;
    int ntaps, Ktot;
    int Ngemm;
    int Ho, Wo, Co;
    int osh, oa, osw, ob;
    int accumulate;
    int vec_out;  // set by launch_igemm: output rows are 16-byte granular (1) or, pipelined bf16 kernel, 8-byte granular (2): vector epilogue
    unsigned src_bytes, wpk_bytes;  // sizes of src and wpk (both below 4 GiB: buffer addressing)
    // Optional per-channel partial sums of the STORED output for a following batch-norm: stats[0][r][n] = sum and
    // stats[1][r][n] = sum of squares over the r-th disjoint share of the rows, r < stats_rows.  Only set when
    // igemm_stats_rows() named the row count for exactly this launch.
    float *stats;
    int stats_rows;
    bool packed;      // wpk was written by the launch before this one (backward-data)
    // Backward-data of a stride-2 layer whose taps all fall into residue class (0, 0): the launch for that class also
    // writes zeros to the other (up to three) pixels of each row's 2x2 output cell.  Only the short-reduction kernel
    // honours it: set it only after conv_pw_applicable() said yes for these arguments.
    int zero_cell;
    // Grouped convolution (groups > 1; 0 or 1 = plain): the launch computes `groups` independent problems of the
    // shape above.  Group g reads channels [g*Cs, (g+1)*Cs) of source pixels that are src_ld channels apart, the filter
    // rows [g*Ngemm, (g+1)*Ngemm) of wpk, and writes columns [g*Ngemm, (g+1)*Ngemm) of the Co-channel output pixels.
    // Only the generic kernel runs such launches; src_ld is ignored (taken as Cs) for plain ones.
    int groups, src_ld;
    short off_h[kMaxTaps];
    short off_w[kMaxTaps];
    // Backward-data straight from the caller's filter (igemm_pipe_gathers said so): element (n, tap t, channel c) lies at
    // w_tap[t] * Ngemm + c * w_sc + n of wpk, where it would be packed to [n][t][c].
    int gather, w_sc;
    unsigned char w_tap[kMaxTaps];
};
int launch_igemm(int dtype, const IgemmArgs &a, hipStream_t stream);
// Rows of partial sums the kernel launch_igemm would pick writes from its epilogue; 0 if that kernel has no
// statistics epilogue (the caller then runs a separate reduction pass).  Host only, depends on the shape alone.
int igemm_stats_rows(int dtype, const IgemmArgs &a);
// every layer whose channel runs are 16-byte granular and that has no kernel of its own (groups, src_ld, vec_out set)
int launch_igemm_pipe(int dtype, const IgemmArgs *a, int count, hipStream_t stream);
int igemm_pipe_stats_rows(int dtype, const IgemmArgs &a);
// the residue classes of a backward-data pass (sizes only are looked at): small enough that the kernel fetches the filter itself
bool igemm_pipe_gathers(int dtype, const IgemmArgs *a, int count);
// the residue classes of one strided backward-data pass (up to four argument sets on the same tensors) in one launch of it; a
// class that no tap reaches (ntaps = 0) is filled with zeros
bool igemm_pipe_multi_applicable(int dtype, const IgemmArgs *a, int count);
int launch_igemm_pipe_multi(int dtype, const IgemmArgs *a, int count, hipStream_t stream);
// bf16 layers with one, two or four taps and at most 256 reduction indices (memory-bound: filter resident in LDS,
// pixels loaded straight into MFMA operand registers)
bool conv_pw_applicable(int dtype, const IgemmArgs &a);
int launch_conv_pw(const IgemmArgs &a, hipStream_t stream);
int conv_pw_stats_rows(const IgemmArgs &a);
// bf16 3x3 stride-1 64->64 special case (filter resident in LDS, input tile staged once with halo)
bool halo64_applicable(int dtype, const IgemmArgs &a);
int launch_halo64(const IgemmArgs &a, hipStream_t stream);
int halo64_stats_rows(const IgemmArgs &a);
// bf16 3x3 stride-1 layers with 128..512 input channels (input rows with halo staged once, filter streamed from L2
// into MFMA operand registers)
bool halo_wide_applicable(int dtype, const IgemmArgs &a);
int launch_halo_wide(const IgemmArgs &a, hipStream_t stream);
int halo_wide_stats_rows(const IgemmArgs &a);
// forward of a 3x3 stride-2 pad-1 layer with 128 or 256 input channels: the same kernel on four parity planes of x
bool halo_wide_fwd_s2_applicable(int dtype, const IgemmArgs &a);
int halo_wide_fwd_s2_stats_rows(const IgemmArgs &a);
int launch_halo_wide_fwd_s2(const IgemmArgs &a, hipStream_t stream);
// the four residue classes of the backward-data pass of a bf16 3x3 stride-2 64 -> 64 layer in one launch of the
// filter-stationary kernel (conv_fs64_s2.hip)
bool fs64_dgrad_s2_applicable(int dtype, const IgemmArgs *a, int count);
int launch_fs64_dgrad_s2(const IgemmArgs *a, int count, hipStream_t stream);
// forward of the same layer (stride 2 as four parity planes of the input), same file
bool fs64_fwd_s2_applicable(int dtype, const IgemmArgs &a);
int fs64_fwd_s2_stats_rows(const IgemmArgs &a);
int launch_fs64_fwd_s2(const IgemmArgs &a, hipStream_t stream);
// the residue classes of one strided backward-data pass of such a layer in one launch, sharing the staged tiles
bool halo_wide_multi_applicable(int dtype, const IgemmArgs *a, int count);
int launch_halo_wide_multi(const IgemmArgs *a, int count, hipStream_t stream);

// fp32 3x3 64 -> 64 layers on images 32 pixels wide, act [2][64]: of relu(act[c]*x + act[64 + c]), applied on load.  Forward (stats: the rows that the
// kernel of the stored activation would leave) and backward-weight (partial sums as wgrad_halo64)
bool halo64_f32_act_applicable(int dtype, const IgemmArgs &a);
int launch_halo64_f32_act(const IgemmArgs &a, const float *act, float *stats, int stats_rows, hipStream_t stream);

// layers with at most four channels on one side (the 3-channel stride-1 image stem): direct kernels, no MFMA
bool tiny_src_applicable(int dtype, const IgemmArgs &a);    // few source channels (forward)
int launch_tiny_src(int dtype, const IgemmArgs &a, hipStream_t stream);
bool tiny_out_applicable(int dtype, const IgemmArgs &a);    // few output channels (backward-data)
int launch_tiny_out(int dtype, const IgemmArgs &a, hipStream_t stream);
// depthwise layers (grouped launches with one channel per group on both sides, channel count a multiple of the vector
// width): direct kernels bound by memory bandwidth, no MFMA
bool depthwise_applicable(int dtype, const IgemmArgs &a);
int launch_depthwise(int dtype, const IgemmArgs &a, hipStream_t stream);

// grouped bf16 3x3 stride-1 layers with eight channels per group on both sides: matrix units, strips of rows in LDS
bool grouped8_applicable(int dtype, const IgemmArgs &a);
int launch_grouped8(const IgemmArgs &a, hipStream_t stream);

// ------------------------------------------------------------------ wgrad
// part[split][k][t][c] = sum over the split's share of rows l = (img, p, q) of
//   dy[img][p][q][k] * x[img][p*sh - ph + off_h[t]][q*sw - pw + off_w[t]][c]
struct WgradArgs {
    const void *x;   // NHWC [Nimg][H][W][C]
    const void *dy;  // NHWC [Nimg][P][Q][K]
    float *part;     // [splits][K][ntaps*C]
    int Nimg, H, W, C, P, Q, K;
    int sh, sw, ph, pw;
    int ntaps;
    int L;           // Nimg*P*Q
    int rows_per_split;  // multiple of the kernel's BK
    int splits;
    // Grouped convolution (groups > 1; 0 or 1 = plain): C and K are the channel counts of ONE group, pixels of x are ldx
    // channels apart and pixels of dy ldy channels; group g reads the channel runs [g*C, (g+1)*C) and [g*K, (g+1)*K)
    // and writes rows [g*K, (g+1)*K) of part[split][groups*K][ntaps*C].  Only the generic kernel runs such launches;
    // ldx and ldy are ignored (taken as C and K) for plain ones.
    int groups, ldx, ldy;
    short off_h[kMaxTaps];
    short off_w[kMaxTaps];
};
int wgrad_rows_per_split(int dtype, int L, int K, int ntapsC, int *splits);
int launch_wgrad(int dtype, const WgradArgs &a, hipStream_t stream);
// the pipelined kernel: channel runs of C and K (of one group) that are 16-byte granular, and no kernel of their own
bool wgrad_pipe_applicable(int dtype, int C, int K, int groups);
int wgrad_pipe_rows_per_split(int dtype, int L, int K, int ntapsC, int groups, int *splits);
int launch_wgrad_pipe(int dtype, const WgradArgs &a, hipStream_t stream);   // groups, ldx, ldy set
// bf16 3x3 stride-1 64->64 special case: one [K][taps][C] partial per block, `partials` of them
bool wgrad_halo64_applicable(int dtype, const WgradArgs &a);
int wgrad_halo64_partials(const WgradArgs &a, int *chunks_per_block);
int launch_wgrad_halo64(const WgradArgs &a, hipStream_t stream);
bool rows32_f32_act_applicable(int dtype, const WgradArgs &a);
int rows32_f32_act_partials(const WgradArgs &a, int *chunks_per_block);
int launch_rows32_f32_act(const WgradArgs &a, const float *act, hipStream_t stream);
// at most four input channels: partial sums in the layout of the generic kernel
bool tiny_wgrad_applicable(int dtype, const WgradArgs &a);
int launch_tiny_wgrad(int dtype, const WgradArgs &a, hipStream_t stream);
// depthwise layers: partial sums in the layout of the generic kernel's grouped launch
bool depthwise_wgrad_applicable(int dtype, const WgradArgs &a);
int launch_depthwise_wgrad(int dtype, const WgradArgs &a, hipStream_t stream);
// grouped bf16 3x3 stride-1 layers with eight channels per group: partial sums in the same layout, splits of its own
bool grouped8_wgrad_applicable(int dtype, const WgradArgs &a);
int grouped8_wgrad_splits(const WgradArgs &a);
int launch_grouped8_wgrad(const WgradArgs &a, hipStream_t stream);
// plain bf16 3x3 stride-1 layers with 16 channels in and out: likewise
bool narrow_wgrad_applicable(int dtype, const WgradArgs &a);
int narrow_wgrad_splits(const WgradArgs &a);
int launch_narrow_wgrad(const WgradArgs &a, hipStream_t stream);
// dw[k*sk + t*st + c*sc] (=|+=) sum_s part[s][k][t][c], k < K, c < C, fixed order; part is [splits][Kp][ntaps][Cp].
int launch_wgrad_reduce(const float *part, float *dw, int splits, int K, int Kp, int ntaps, int C, int Cp,
                        long sk, long st, long sc, int accumulate, hipStream_t stream);

// The same for many layers whose dw lies as their partial sums do (`total` outputs), in one launch; sums as above, bit by bit.
struct ReduceItem {
    const float *part;
    float *dw;
    int splits, total, kind, first_block;   // kind, first_block: set by the launcher
};
int launch_wgrad_reduce_many(ReduceItem *items, int count, int accumulate, hipStream_t stream);

// ------------------------------------------------------------------ image stem
// Stride-2 odd square filter with "same" padding on at most 4 input channels and even H, W: all three
// passes run on a space-to-depth copy of the image (16 channels, stride 1).  `ws` must hold
// stem_workspace_bytes(g, pass) bytes.
bool stem_applicable(const ConvGeo &g);
size_t stem_workspace_bytes(const ConvGeo &g, int pass);
// stats / stats_rows: as in IgemmArgs (nullptr: none); *y_nhwc receives the NHWC result (y itself, or its workspace
// copy for NCHW descriptors)
int stem_fwd(const ConvGeo &g, const void *x, const void *w, void *y, char *ws, float *stats, int stats_rows,
             void **y_nhwc, hipStream_t stream);
int stem_stats_rows(const ConvGeo &g);
int stem_dgrad(const ConvGeo &g, const void *dy, const void *w, void *dx, int accumulate, char *ws, hipStream_t stream);
int stem_wgrad(const ConvGeo &g, const void *x, const void *dy, float *dw, int accumulate, char *ws, hipStream_t stream);

// 7x7 stem (4x4 coarse taps), bf16, 64 output channels: forward / backward-data on the space-to-depth grid
bool stem_halo_applicable(int dtype, int U, int K, int Nimg, int H, int W);
int launch_stem_halo(int backward, const void *src, const void *wpk, void *out, int Nimg, int H, int W, float *stats,
                     int stats_rows, hipStream_t stream);
int stem_halo_stats_rows(int Nimg, int H, int W);

// ------------------------------------------------------------------ layout helpers
// dst NHWC with Cp >= C channels per pixel (those from C on are zeros) <- src NCHW.
int launch_nchw_to_nhwc(int dtype, const void *src, void *dst, int N, int C, int H, int W, int Cp,
                        hipStream_t stream);
// dst [rows][Cp] <- src [rows][C], zeros from C on; Cp elements are a multiple of 16 bytes.
int launch_pad_channels(int dtype, const void *src, void *dst, long rows, int C, int Cp, hipStream_t stream);
// dst NCHW (=|+=) src NHWC.
int launch_nhwc_to_nchw(int dtype, const void *src, void *dst, int N, int C, int H, int W,
                        int accumulate, hipStream_t stream);
// out[n][t][c] = w[n*sn + tap_off[t] + c*sc] for n < Nn, t < ntaps, c < Cr, and 0 for Cr <= c < Cs.
int launch_pack_filter(int dtype, const void *w, void *out, int Nn, int ntaps, int Cs, int Cr, long sn,
                       long sc, const int *tap_off_host, hipStream_t stream);
// The same for up to four tap subsets of one filter in one launch, out[k][..][n][t][c] with ntaps[k] taps tap_off_host[k][.],
// and for `groups` filters that lie w_gstep elements apart in w: out[k][g][n][t][c] = w[g*w_gstep + n*sn + ...].
int launch_pack_filters_grouped(int dtype, int count, const void *w, void *const *out, int Nn, const int *ntaps, int Cs, int Cr,
                                long sn, long sc, const int (*tap_off_host)[kMaxTaps], int groups, long w_gstep,
                                hipStream_t stream);

// Small filters of many layers in one launch: out[n][t][c] = w[n*sn + tap_off[t] + c*sc], n < Nn, t < ntaps, c < Cs.
struct PackItem {
    const void *w;
    void *out;
    int Nn, ntaps, Cs, sn, sc, first_block;
    int tap_off[9];
};
int launch_pack_many(int dtype, PackItem *items, int count, hipStream_t stream);   // sets first_block; any count

// out[img][i*osh + oa][j*osw + ob][0..Co) = 0 for i < Mi, j < Mj (NHWC).
int launch_zero_class(int dtype, void *out, int Nimg, int Ho, int Wo, int Co, int Mi, int Mj, int osh, int oa, int osw,
                      int ob, hipStream_t stream);

// ------------------------------------------------------------------ batch-norm, pooling
int bn_partial_blocks(const nsk_bn_desc_t &d);
size_t bn_mask_bytes(const nsk_bn_desc_t &d);
int launch_bn_fwd(const nsk_bn_desc_t &d, const void *x, const void *residual, const float *gamma,
                  const float *beta, void *out, float *save_mean, float *save_invstd,
                  float *running_mean, float *running_var, void *ws, unsigned char *relu_mask, const float *stats,
                  int stats_rows, hipStream_t stream);
int bn_stats_rows(const nsk_bn_desc_t &d);
int launch_bn_stats(const nsk_bn_desc_t &d, const void *x, float *stats, int rows, hipStream_t stream);   // any number of rows
int launch_bn_bwd(const nsk_bn_desc_t &d, const void *x, const void *out, const void *dout,
                  const float *gamma, const float *save_mean, const float *save_invstd, void *dx,
                  void *dres, float *dgamma, float *dbeta, void *ws, const unsigned char *relu_mask,
                  hipStream_t stream, const float *act = nullptr);
// The normalised activation applied by its consumers on load (scale and shift per channel: coeffs = [2][C] floats)
bool bn_act_supported(const nsk_bn_desc_t &d);
int launch_bn_coeffs(const nsk_bn_desc_t &d, const float *gamma, const float *beta, const float *stats, int stats_rows,
                     float *save_mean, float *save_invstd, float *running_mean, float *running_var, float *coeffs,
                     void *ws, hipStream_t stream);
int launch_bn_act(const nsk_bn_desc_t &d, const void *x, const float *coeffs, void *out, hipStream_t stream);
int launch_maxpool_fwd(const nsk_pool_desc_t &d, int P, int Q, const void *x, void *y,
                       signed char *idx, hipStream_t stream);
int launch_maxpool_bwd(const nsk_pool_desc_t &d, int P, int Q, const void *dy,
                       const signed char *idx, void *dx, hipStream_t stream);

}  // namespace nsk
