// Implicit-GEMM convolution for every layer without a kernel of its own whose channel runs are 16-byte granular
// (forward, backward-data, grouped launches; fp32 and bf16): the pipelined tile kernel.
//
// GEMM view: rows m = output pixels, columns n = output channels, reduction k = (filter tap, input channel).
//
// What bounds it: a k-tile is 128 bytes of the reduction index for BM + BN rows.  With one k-tile in flight per block
// (register prefetch, one barrier) a 128 x 128 bf16 tile took 2000 clocks per k-tile, of which the matrix units need
// 512: the rest was the latency of the loads, because layers with few output pixels (7x7 images) give a CU one block
// only.  Here the operands go from memory straight into LDS (16 bytes per lane, no registers), ST k-tiles deep, and a
// k-tile costs one counted wait and one barrier.
//
// Layout in LDS: rows of 128 bytes, the eight 16-byte pieces of row r stored at piece ^ ((r >> 1) & 7), so that the
// sixteen rows a fragment read serves at once cover all 64 banks.  A direct load writes 64 consecutive 16-byte slots
// (eight rows), so the exchange is made in the source address: a lane always fetches the same piece of its rows.
//
// Small problems: the block's four wavefronts are WM x WN x WK; with WK > 1 the wavefronts of a group multiply
// different parts of each k-tile and their sums are added through LDS in a fixed order, so that a 32 x 32 tile still
// keeps four wavefronts busy.
//
// Output rows of whole 8-byte vectors (bf16, channels 4 past a multiple of 8) are staged like the others and stored in
// halves: bf16 104 -> 100 at 28x28, N=32 18.6 -> 13.0 us against element-wise stores, 1x1 12 -> 36 at 56x56, N=64 40.5 -> 23.3.
//
// Measured against the one-tile-ahead kernel (us, forward): bf16 3x3 512->512 at 7x7, N=64 77.7 -> 27.2; fp32 3x3 72->100
// at 29x37, N=20 80.8 -> 43.9 (and 36 on pieces, see the tiles); fp32 3x3 16->16 at 32x32, N=8 16.8 -> 5.7.  Without the exchange of pieces the first takes
// 64 us (bank conflicts).
#include <limits.h>

#include "nsk_internal.h"

namespace nsk {
namespace {

template <typename T> struct PipeTraits;
template <> struct PipeTraits<float> {
    static constexpr int VEC = 4;
    typedef f32x4 Vec;
};
template <> struct PipeTraits<bf16_t> {
    static constexpr int VEC = 8;
    typedef bf16x8 Vec;
};

__device__ inline float to_f(float v) { return v; }
__device__ inline float to_f(bf16_t v) { return (float)v; }

typedef __attribute__((address_space(3))) void lds_void;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int PK_BYTES = 128;   // bytes of reduction index per k-tile row

constexpr int kMaxProblems = 4;
template <int NP> struct PipeProblems {   // NP = 1 or kMaxProblems: a plain launch carries 400 bytes of arguments, not 1.7 KB
    IgemmArgs a[NP];
    int tiles_m[NP];
    int cols[NP];      // the tiles of one column block follow each other, not those of one row block
    Div by[NP];        // tiles_m or tiles_n accordingly
    int tiles_n;
};

// GATHER: the filter is fetched as the caller holds it (IgemmArgs::gather), four bytes a lane.
template <typename T, int BM, int BN, int WM, int WN, int WK, int ST, int NP, bool GATHER>
__global__ __launch_bounds__(64 * WM * WN * WK, sizeof(T) == 4 && BM * BN >= 4096 ? 2 : 1) void igemm_pipe_kernel(const PipeProblems<NP> pp)
{
    const int prob = NP > 1 ? blockIdx.y : 0;   // (the problems of a launch differ in their pixels and taps)
    const IgemmArgs &a = pp.a[prob];
    const int tiles_m = pp.tiles_m[prob], tiles_n = pp.tiles_n;
    if ((int)blockIdx.x >= tiles_m * tiles_n) return;
    typedef typename PipeTraits<T>::Vec Vec;
    constexpr int VEC = PipeTraits<T>::VEC, ES = (int)sizeof(T), BK = PK_BYTES / ES;
    constexpr int NW = WM * WN * WK;                    // wavefronts per block
    static_assert((NW == 4 || NW == 8) && BM <= 64 * NW, "four or eight wavefronts per block");
    constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    constexpr int RA = BM / 8 / NW, RB = BN / 8 / NW;           // direct loads per wavefront and k-tile (eight rows each)
    constexpr int LOADS = RA + (GATHER ? 4 : 1) * RB;
    static_assert(!GATHER || ES == 4, "one element a load");
    constexpr int TA = BM * PK_BYTES, TB = BN * PK_BYTES;
    constexpr int SROW = 32 * ES + 16;                  // epilogue: staged bytes per pixel (padded)
    constexpr int STRIPS = WM * WN * 32 * SROW, SUMS = WM * WN * (WK - 1) * FN * 4096;   // SUMS: of the wavefronts wk > 0
    constexpr int EPI = STRIPS > SUMS ? STRIPS : SUMS, TA0 = TA > EPI ? TA : EPI;
    static_assert(ST >= 2 && ST <= 4, "stages");
    constexpr bool SPLIT = ES == 4 && BM * BN >= 4096;   // fp32 products of bf16 pieces (small tiles make too little of each piece)
    static_assert(!SPLIT || WK <= 2, "a k-tile of fp32 is two groups of 16");

    // one variable per stage and operand: the compiler keeps the reads of one apart from the direct loads into the others
    __shared__ __attribute__((aligned(1024))) unsigned char sa0[TA0], sa1[TA], sa2[ST > 2 ? TA : 16], sa3[ST == 4 ? TA : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sb0[TB], sb1[TB], sb2[ST > 2 ? TB : 16], sb3[ST == 4 ? TB : 16];
    __shared__ unsigned s_base[BM], s_out[BM];   // byte offsets of a row's base pixel in src and of its pixel in out (~0: none)
    __shared__ int s_bh[BM], s_bw[BM];
    __shared__ int s_oh[kMaxTaps], s_ow[kMaxTaps];
    __shared__ unsigned s_delta[kMaxTaps];
    __shared__ unsigned s_wtap[GATHER ? kMaxTaps : 1];
#define NSK_STAGE(S, P) ((S) == 0 ? P##0 : (S) == 1 ? P##1 : (S) == 2 ? P##2 : P##3)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / (WK * WN);

    // Tiles of one row block on one XCD, next to each other (blocks go to the eight XCDs in turn): its L2 then holds
    // the activation rows they share.  Where the filter is the larger operand, tiles of one column block: an XCD then reads
    // its columns' filter and all of src instead of the whole filter (3x3 on 7x7 images, rows / columns first, us: 1024
    // channels, 8 images 40.9 / 33.3 forward; 512 channels, 8 .. 16 images 22.4 / 16.5 forward, 29.2 / 20.8 backward-data;
    // 32 images 22.6 / 20.2, 29.1 / 23.0; 64 images, filter 1.5 times src, 29.2 / 29.5, 33.9 / 31.8), while src fits an L2 of 4 MB (1024 -> 512, 64
    // images of 7x7, 6.4 MB, 45.9 / 55.0; 1024 -> 1024, 128 images, 114.9 / 123.3).  Order and divisor come from the host: found
    // here, with a division, they were 5% of a launch of many short blocks (backward-data of 16 -> 16 3x3 stride 2, 256 images of 32x32,
    // 17.4 us; the division by tiles_n alone, without the second order, 16.4; this 16.2).
    int bm, bn;
    {
        const int total = tiles_m * tiles_n, x = blockIdx.x & 7;
        const int q = total >> 3, r = total & 7;
        const int t = x * q + min(x, r) + ((int)blockIdx.x >> 3);
        const bool cols = pp.cols[prob] != 0;
        const int n = cols ? tiles_m : tiles_n, o = divide(t, pp.by[prob]), i = t - o * n;
        bm = cols ? i : o;
        bn = cols ? o : i;
    }
    const int m0 = bm * BM, n0 = bn * BN;
    const int grp = blockIdx.z, ld = a.src_ld;
    const int src_c0 = grp * a.Cs;
    const long wrow0 = (long)grp * a.Ngemm;

    if (tid < kMaxTaps) {
        const int oh = a.off_h[tid], ow = a.off_w[tid];
        s_oh[tid] = oh;
        s_ow[tid] = ow;
        s_delta[tid] = (unsigned)((oh * a.Ws + ow) * ld * ES);
        if constexpr (GATHER) s_wtap[tid] = (unsigned)a.w_tap[tid] * (unsigned)(a.Ngemm * ES);
    }
    if (tid < BM) {
        const int m = m0 + tid, per_img = a.Mi * a.Mj;
        const int img = m / per_img, rem = m - img * per_img, i = rem / a.Mj, j = rem - i * a.Mj;
        const int bh = i * a.mult_h + a.add_h, bw = j * a.mult_w + a.add_w;
        s_bh[tid] = m < a.M ? bh : INT_MIN / 2;      // (no tap brings such a row into the image)
        s_bw[tid] = bw;
        s_base[tid] = (unsigned)(((((long)img * a.Hs + bh) * a.Ws + bw) * ld + src_c0) * (long)ES);
        s_out[tid] = m < a.M ? (unsigned)(((((long)img * a.Ho + (i * a.osh + a.oa)) * a.Wo + (j * a.osw + a.ob)) * a.Co + wrow0) * ES)
                             : ~0u;
    }
    __syncthreads();

    // This lane's rows of the activation tile: byte offset of the row's base pixel and one bit per tap, set where the tap leaves the image.
    // (Two words, not one of 64 bits: a 64-bit shift whose amount lies in the last register that the kernel has gives wrong bits on this chip,
    // 0.13 of v_lshrrev_b64 by v63 of 64 registers; the masks here came out wrong that way.)
    const int lr = lane >> 3;
    const int piece = (lane & 7) ^ ((wave & 1) * 4 + (lr >> 1));
    unsigned a_base[RA];
    unsigned a_out[RA], a_out_hi[RA];                // taps 0..31, 32..63
    {
        int bh[RA], bw[RA];
#pragma unroll
        for (int u = 0; u < RA; ++u) {
            const int row = 8 * (wave + NW * u) + lr;
            a_base[u] = s_base[row];
            bh[u] = s_bh[row];
            bw[u] = s_bw[row];
            a_out[u] = a_out_hi[u] = 0;
        }
#pragma unroll 1
        for (int t = 0; t < a.ntaps; ++t) {
            const int oh = s_oh[t], ow = s_ow[t];
#pragma unroll
            for (int u = 0; u < RA; ++u) {
                const bool in = (unsigned)(bh[u] + oh) < (unsigned)a.Hs & (unsigned)(bw[u] + ow) < (unsigned)a.Ws;
                const unsigned bit = in ? 0u : 1u << (t & 31);
                a_out[u] |= t < 32 ? bit : 0u;
                a_out_hi[u] |= t < 32 ? 0u : bit;
            }
        }
    }
    unsigned b_row[RB], b_bad[RB];
    const __amdgpu_buffer_rsrc_t src_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.src, 0, a.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wpk_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.wpk, 0, a.wpk_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t out_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        a.out, 0, (unsigned)((long)a.Nimg * a.Ho * a.Wo * a.Co * ES), 0x00020000);

    // position of this lane's piece inside (tap, channel), of the next k-tile to be requested; a k-tile further is
    // q_tap taps and r_c channels
    const int q_tap = BK / a.Cs, r_c = BK - q_tap * a.Cs;
    int cur_tap, cur_c;
    // GATHER: of every eight rows a load brings two, dword by dword as they will lie, so a lane's reduction index differs from load to load
    int g_tap[GATHER ? 4 : 1], g_c[GATHER ? 4 : 1];
    auto start_requests = [&]() {
        cur_tap = piece * VEC / a.Cs;
        cur_c = piece * VEC - cur_tap * a.Cs;
        if constexpr (GATHER) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = ((((lane >> 2) & 7) ^ ((wave & 1) * 4 + q)) * 4) + (lane & 3);
                g_tap[q] = k / a.Cs;
                g_c[q] = k - g_tap[q] * a.Cs;
            }
        }
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int n = n0 + 8 * (wave + NW * u) + lr;
            b_row[u] = (unsigned)((wrow0 + n) * a.Ktot * (long)ES) + (unsigned)(piece * 16);
            b_bad[u] = n < a.Ngemm ? 0u : ~0u;
        }
    };
    // Offsets are made out of range (reads: zeros, writes: dropped) with bit operations: a branch around a direct load
    // would split it in two.
    auto request = [&](auto S) {
        constexpr int I = S.value;
        const unsigned k_bad = (unsigned)((a.ntaps - 1 - cur_tap) >> 31);
        const int tap = cur_tap & (kMaxTaps - 1);
        const unsigned delta = s_delta[tap] + (unsigned)(cur_c * ES);
#pragma unroll
        for (int u = 0; u < RA; ++u) {
            const unsigned bad = (unsigned)__builtin_amdgcn_sbfe((int)(tap & 32 ? a_out_hi[u] : a_out[u]), (unsigned)tap & 31u, 1u);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(src_rsrc, (lds_void *)&NSK_STAGE(I, sa)[(wave + NW * u) * 1024], 16,
                                                     (int)((a_base[u] + delta) | bad | k_bad), 0, 0, 0);
        }
        if constexpr (GATHER) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned bad_k = (unsigned)((a.ntaps - 1 - g_tap[q]) >> 31);
                const unsigned at = s_wtap[g_tap[q] & (kMaxTaps - 1)] + (unsigned)(g_c[q] * a.w_sc * ES);
#pragma unroll
                for (int u = 0; u < RB; ++u) {
                    const int n = n0 + 8 * (wave + NW * u) + 2 * q + (lane >> 5);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wpk_rsrc, (lds_void *)&NSK_STAGE(I, sb)[(wave + NW * u) * 1024 + q * 256], 4,
                                                             (int)((at + (unsigned)(n * ES)) | bad_k | (n < a.Ngemm ? 0u : ~0u)), 0, 0, 0);
                }
                g_c[q] += r_c;
                g_tap[q] += q_tap;
                const bool w = g_c[q] >= a.Cs;
                g_c[q] -= w ? a.Cs : 0;
                g_tap[q] += w ? 1 : 0;
            }
        }
#pragma unroll
        for (int u = 0; u < (GATHER ? 0 : RB); ++u) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wpk_rsrc, (lds_void *)&NSK_STAGE(I, sb)[(wave + NW * u) * 1024], 16,
                                                     (int)(b_row[u] | b_bad[u] | k_bad), 0, 0, 0);
            b_row[u] += PK_BYTES;
        }
        cur_c += r_c;
        cur_tap += q_tap;
        const bool wrap = cur_c >= a.Cs;
        cur_c -= wrap ? a.Cs : 0;
        cur_tap += wrap ? 1 : 0;
    };

    // The filter rows are the MFMA "A" operand and the pixels the "B" operand, so a lane ends up with 4 consecutive
    // channels of one pixel per accumulator quad: acc[mi][ni][4g+j] is channel 32*ni + 8*g + 4*(lane/32) + j of pixel
    // 32*mi + lane%32 of the wavefront's sub-tile.
    const int frow = lane & 31, fk = lane >> 5, fsw = (frow >> 1) & 7;
    T *__restrict__ out = (T *)a.out;
    const int wcol0 = n0 + wn * (FN * 32), wrow = wm * (FM * 32);
    f32x16 acc[FM][FN], lo[FM][FN];    // lo: of the smaller products
    auto start_sums = [&](float scale) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
        if (a.accumulate && a.vec_out && wk == 0) {
            // start from the old values: the sum is then rounded to the storage type exactly once
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) {
                const unsigned off = s_out[wrow + mi * 32 + frow], off_bad = off == ~0u ? ~0u : 0u;
#pragma unroll
                for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int col = wcol0 + ni * 32 + g * 8 + fk * 4;
                        const int at = (int)((off + (unsigned)(col * ES)) | off_bad | (col < a.Ngemm ? 0u : ~0u));
                        if constexpr (ES == 2) {
                            const bf16x4 v = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(out_rsrc, at, 0, 0));
#pragma unroll
                            for (int j = 0; j < 4; ++j) acc[mi][ni][g * 4 + j] = (float)v[j];
                        } else {
                            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(out_rsrc, at, 0, 0));
#pragma unroll
                            for (int j = 0; j < 4; ++j) acc[mi][ni][g * 4 + j] = v[j] * scale;
                        }
                    }
            }
        }
    };

    const int nk = (a.Ktot + BK - 1) / BK;
    // PIECES: fp32 products of bf16 pieces
    auto multiply = [&](auto PIECES, auto S) {
        constexpr int I = S.value;
        const int oa = (wrow + frow) * PK_BYTES, ob = (wn * (FN * 32) + frow) * PK_BYTES;
        if constexpr (decltype(PIECES)::value) {
            // lane (row, half) holds two 16-byte pieces of a group of 16, the same two of both operands
#pragma unroll
            for (int i = 0; i < 2 / WK; ++i) {
                const int g = wk * (2 / WK) + i, at0 = ((g * 4 + fk) ^ fsw) * 16, at1 = ((g * 4 + 2 + fk) ^ fsw) * 16;
                auto split = [&](const unsigned char *row) {
                    const f32x4 u = *(const f32x4 *)(row + at0), v = *(const f32x4 *)(row + at1);
                    const float x[8] = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
                    return split3(x);
                };
                Pieces pa[FM], pb[FN];
#pragma unroll
                for (int mi = 0; mi < FM; ++mi) pa[mi] = split(&NSK_STAGE(I, sa)[oa + mi * 32 * PK_BYTES]);
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) pb[ni] = split(&NSK_STAGE(I, sb)[ob + ni * 32 * PK_BYTES]);
                multiply_pieces<true>(pb, pa, acc, lo);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < 4 / WK; ++i) {
            const int ks = wk * (4 / WK) + i, at = (((ks * 2 + fk) ^ fsw) * 16);
            Vec af[FM], bfv[FN];
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) af[mi] = *(const Vec *)&NSK_STAGE(I, sa)[oa + at + mi * 32 * PK_BYTES];
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) bfv[ni] = *(const Vec *)&NSK_STAGE(I, sb)[ob + at + ni * 32 * PK_BYTES];
            if constexpr (ES == 2) {
#pragma unroll
                for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < FN; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfv[ni], af[mi], acc[mi][ni], 0, 0, 0);
            } else {
                // lane (row, half) holds k = 4*half + t of this group of 8, the same map for both operands
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                        for (int ni = 0; ni < FN; ++ni)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(bfv[ni][t], af[mi][t], acc[mi][ni], 0, 0, 0);
            }
        }
    };
    auto products = [&](auto PIECES) {
        start_requests();
        start_sums(decltype(PIECES)::value ? kSumScale : 1.f);
        static_for<0, ST - 1>([&](auto S) { request(S); });   // (k-tiles past the end are requested out of range: zeros)
        // The loop body is ST steps without a branch, the remainder follows: where a step could leave the loop, the compiler
        // would take the stage requested last for one that the first step reads, and wait for it.
#define NSK_STEP(S)                                                                                              \
    wait_vm<(ST - 2) * LOADS>();  /* this wavefront's part of the k-tile has arrived */                          \
    __builtin_amdgcn_s_barrier(); /* everybody's has, and nobody reads the stage requested next any more */      \
    asm volatile("" ::: "memory");                                                                               \
    request(std::integral_constant<int, ((S) + ST - 1) % ST>{});                                                 \
    multiply(PIECES, std::integral_constant<int, (S)>{});
        for (int n = nk / ST; n > 0; --n) {
            NSK_STEP(0)
            NSK_STEP(1)
            if constexpr (ST > 2) {
                NSK_STEP(2)
            }
            if constexpr (ST == 4) {
                NSK_STEP(3)
            }
        }
#undef NSK_STEP
        // (the last ST - 1 k-tiles have been requested; what the loop requested past the end were zeros)
#define NSK_REST(S)                             \
    wait_vm<(ST - 2 - (S) > 0 ? ST - 2 - (S) : 0) * LOADS>();          \
    __builtin_amdgcn_s_barrier();               \
    asm volatile("" ::: "memory");              \
    multiply(PIECES, std::integral_constant<int, (S)>{});
        const int rest = nk % ST;
        if (rest > 0) {
            NSK_REST(0)
        }
        if constexpr (ST > 2) {
            if (rest > 1) {
                NSK_REST(1)
            }
        }
        if constexpr (ST == 4) {
            if (rest > 2) {
                NSK_REST(2)
            }
        }
#undef NSK_REST
        wait_vm<0>();          // (requests past the end still write zeros into LDS)
    };
    if constexpr (SPLIT) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) lo[mi][ni][v] = 0.f;
    }
    products(std::integral_constant<bool, SPLIT>{});
    if constexpr (SPLIT) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] = (acc[mi][ni][v] + lo[mi][ni][v]) * (1.f / kSumScale);
        if (__syncthreads_or(!finite_sums(acc))) products(std::integral_constant<bool, false>{});
    }
    __syncthreads();

    if constexpr (WK > 1) {
        // add the wavefronts of a group in a fixed order, one row of accumulator tiles at a time
        float *red = (float *)sa0;
        const int slot = (wm * WN + wn) * (WK - 1);
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
            if (mi > 0) __syncthreads();
            if (wk > 0) {
#pragma unroll
                for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; v += 4)
                        *(f32x4 *)(red + (((slot + wk - 1) * FN + ni) * 4 + v / 4) * 256 + lane * 4) =
                            f32x4{acc[mi][ni][v], acc[mi][ni][v + 1], acc[mi][ni][v + 2], acc[mi][ni][v + 3]};
            }
            __syncthreads();
            if (wk > 0) continue;
            // (0 + 1) + (2 + 3): two roundings deep, not three
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; v += 4) {
                    f32x4 p[WK];
#pragma unroll
                    for (int w = 1; w < WK; ++w)
                        p[w] = *(const f32x4 *)(red + (((slot + w - 1) * FN + ni) * 4 + v / 4) * 256 + lane * 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc[mi][ni][v + j] += p[1][j];
                        if constexpr (WK == 4) acc[mi][ni][v + j] += p[2][j] + p[3][j];
                    }
                }
        }
        __syncthreads();       // (the strips below lie where the sums were)
        if (wk > 0) return;
    }

    if (a.vec_out) {
        // Round to the storage type, transpose one 32 x 32 accumulator tile at a time through this wavefront's strip of
        // the (now idle) first stage, and store 16 contiguous bytes per lane.
        typedef T T4 __attribute__((ext_vector_type(4)));
        constexpr int CPP = 32 * ES / 16;               // 16-byte chunks per pixel
        unsigned char *my_st = sa0 + (wm * WN + wn) * (32 * SROW);
        // Statistics epilogue (forward with a batch-norm behind it): a lane always reads back the same 16-byte piece
        // (VEC channels) of each staged row, so it adds those channels up over all the rows it stores; one cross-lane
        // reduction per block and at most two rows of partial sums.  With every value added across all lanes by itself
        // (64 exchanges per 32 channels, now 15) 256 -> 1024 1x1 on 25 k pixels took 45 us with statistics and 34 without.
        float ssum[FN][VEC], ssq[FN][VEC];
#pragma unroll
        for (int ni = 0; ni < FN; ++ni)
#pragma unroll
            for (int e = 0; e < VEC; ++e) ssum[ni][e] = ssq[ni][e] = 0.f;
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    T4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j) pk[j] = (T)acc[mi][ni][g * 4 + j];
                    *(T4 *)(my_st + frow * SROW + (g * 8 + fk * 4) * ES) = pk;
                }
#pragma unroll
                for (int jj = 0; jj < 32 * CPP / 64; ++jj) {
                    const int idx = lane + 64 * jj, pos = idx / CPP, ck = idx % CPP;
                    const Vec v = *(const Vec *)(my_st + pos * SROW + ck * 16);
                    const unsigned off = s_out[wrow + mi * 32 + pos];
                    const int col = wcol0 + ni * 32 + ck * VEC;
                    const unsigned bad = (off == ~0u ? ~0u : 0u) | (col < a.Ngemm ? 0u : ~0u);
                    const unsigned at = (off + (unsigned)(col * ES)) | bad;
                    if (ES == 2 && a.vec_out == 2) {   // rows of whole 8-byte vectors: the last piece may be half one
                        const u32x4 q = __builtin_bit_cast(u32x4, v);
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{q[0], q[1]}, out_rsrc, (int)at, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{q[2], q[3]}, out_rsrc, (int)((at + 8u) | bad | (col + 4 < a.Ngemm ? 0u : ~0u)), 0, 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out_rsrc, (int)at, 0, 0);
                    }
                    if (a.stats) {
                        u32x4 q = __builtin_bit_cast(u32x4, v);
#pragma unroll
                        for (int e = 0; e < 4; ++e) q[e] &= ~bad;
                        const Vec kept = __builtin_bit_cast(Vec, q);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            const float f = to_f(kept[e]);
                            ssum[ni][e] += f;
                            ssq[ni][e] += f * f;
                        }
                    }
                }
            }
        if (a.stats) {
            // (VEC channels' sums and squares over the 64 / CPP lanes of a piece: as many values as lanes)
            static_assert(2 * VEC * CPP == 64, "a value a lane");
            static_assert(WM * WN * FN * 256 <= TB, "inside a stage");
            static_assert(WM == 1 || WM == 2 || WM == 4, "wavefront rows");
            // Four wavefront rows are added through LDS, in fp64, and leave two rows, the sum and what rounding it cuts off: as exact as a row
            // each, half as many for the batch-norm behind to read.  (One rounded row moved means by up to 0.4 of their error against 64 bits.)
            float *part = (float *)sb0 + lane;
            float mine[FN];
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
                float v[2 * VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    v[i] = ssum[ni][i];
                    v[VEC + i] = ssq[ni][i];
                }
                fold_lanes<CPP>(v);
                mine[ni] = v[0];
                if (WM == 4 && wm > 0) part[((wm * WN + wn) * FN + ni) * 64] = v[0];
            }
            if constexpr (WM == 4) {
                lds_barrier();
                if (wm > 0) return;
            }
            const int e = lane / CPP % VEC, row = WM == 4 ? 2 * bm : bm * WM + wm;
            float *r = a.stats + ((size_t)(lane / 32) * a.stats_rows + row) * a.Ngemm;
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
                const int col = wcol0 + ni * 32 + lane % CPP * VEC + e;
                if constexpr (WM == 4) {
                    double sum = mine[ni];
#pragma unroll
                    for (int w = 1; w < WM; ++w) sum += (double)part[((w * WN + wn) * FN + ni) * 64];
                    mine[ni] = (float)sum;
                    if (col < a.Ngemm) r[a.Ngemm + col] = mine[ni] - mine[ni] == 0.f ? (float)(sum - (double)mine[ni]) : 0.f;
                }
                if (col < a.Ngemm) r[col] = mine[ni];
            }
        }
    } else {
        // element-wise stores (output rows that are not made of vectors)
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
            const unsigned off_b = s_out[wrow + mi * 32 + frow];
            if (off_b == ~0u) continue;
            const long off = off_b / ES;
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int col = wcol0 + ni * 32 + 8 * (v >> 2) + 4 * fk + (v & 3);
                    if (col < a.Ngemm) {
                        float r = acc[mi][ni][v];
                        if (a.accumulate) r += to_f(out[off + col]);
                        out[off + col] = (T)r;
                    }
                }
        }
    }
}

// Tile shapes with what a launch of them costs (us): `fixed` + the larger of whole rounds of blocks on the 256 CUs, a block
// costing `step` a k-tile and `rest` once, and `per_mb` a megabyte moved (what one or two blocks a CU keep on their way).
// `stats` and 1.5 ns a row of them are what the statistics add, in the epilogue and in the batch-norm that reads them.
// Fitted to 900 bf16 passes of 1x1 and 3x3 filters, stride 1 and 2, 16 to 2048 channels, 0.5 k to 400 k pixels, each timed with
// every shape: the choice is on average 0.7% off the best shape and 5% in the worst twentieth (with the clocks of a block
// alone and no bound on the bytes 2% and 14%: 1x1 layers whose last round was nearly empty took up to 1.5 times the time
// of the best one, 64 -> 128 on 38 k pixels 9.0 us instead of 6.1).
// bf16 is bound by the fill of LDS: eight wavefronts per block bring 38-42 B/clk into a CU, four only 31, so all bf16 shapes
// but the narrowest have eight.  128 x 64 has three stages, not four, where there are blocks enough to put two on a CU, which
// fill while the other stores (median over those layers 0.76 of its time; 128 -> 64 on 75 k pixels 10.0 -> 7.5 us,
// 256 -> 128 on 200 k 50 -> 35).
// fp32: tiles of 4096 outputs and more multiply bf16 pieces (nsk_internal.h), bound by the vector unit that makes them, so the sub-tile of a
// wavefront is 64 x 64 or 64 x 32; smaller tiles, for layers that leave CUs idle otherwise, run on the fp32 matrix unit (256 clocks per 32 x 32
// and k-tile).  Fitted to 260 forward passes of the same ranges: the choice is on average 1.8% off the best shape, 10% in the worst twentieth.
// Forward, fp32 unit only / this, us: 3x3 64 -> 64 at 56x56, N=64 154 / 119; 128 -> 128 at 28x28, N=64 147 / 112; 72 -> 100 at 29x37,
// N=20 44 / 36; 1x1 256 -> 768 on 10 k pixels 50 / 32; error against 64 bits 3.0e-7 / 1.0e-7, 4.2e-7 / 2.0e-7, 3.2e-7 / 1.0e-7, 2.1e-7 / 0.9e-7.
struct PipeTile {
    int bm, bn, rows, wk;      // rows: of statistics; wk: parts a k-tile's sums are made in
    double step, rest, fixed, per_mb, stats;
};
constexpr PipeTile kTilesBf16[] = {{256, 128, 2, 1, 0.827, 4.71, 0.99, 0.017, 1.4}, {128, 128, 2, 1, 0.494, 3.15, 1.3, 0.219, 0},
                                   {256, 64, 2, 1, 0.587, 3.34, 0.92, 0.217, 0},    {128, 64, 2, 1, 0.302, 1.47, 2.96, 0.074, 0},
                                   {64, 64, 2, 2, 0.224, 2.12, 1.25, 0.251, 0},     {128, 32, 2, 1, 0.30, 0.9, 2.34, 0.162, 0},
                                   {128, 128, 2, 1, 0, 0, 1e9, 0, 0}};   // kShort (taken by a rule, see cheapest)
constexpr int kShort = 6;
constexpr int kSmallest = 5;
constexpr PipeTile kTilesF32[] = {{128, 64, 2, 2, 0.770, 1.96, 4.79, 0.238, 0}, {64, 64, 1, 2, 0.563, 0, 5.08, 0.361, 0},
                                  {256, 128, 2, 1, 2.19, 6.83, 0, 0.039, 0},    {128, 32, 2, 1, 0.557, 1.01, 4.03, 0.255, 0},
                                  {64, 32, 2, 2, 0.322, 0.73, 3.76, 0.258, 0},  {32, 32, 1, 4, 0.172, 0.68, 3.98, 0.23, 0}};

long block_count(const PipeTile &t, const IgemmArgs *a, int count)
{
    long blocks = 0;
    for (int j = 0; j < count; ++j) blocks += (long)ceil_div(a[j].M, t.bm) * ceil_div(a[j].Ngemm, t.bn);
    return blocks * (a[0].groups > 1 ? a[0].groups : 1);
}

// stats: the launch leaves statistics.  Its shape then makes every sum in the same order as the one without would, so that the
// output does not depend on whether they are asked for.
template <int N> int cheapest(const PipeTile (&tiles)[N], int es, const IgemmArgs *a, int count, bool stats)
{
    const int forced = hooks().igemm_tile;   // NSK_IGEMM_TILE = 1.. (test hook)
    if (forced >= 1) return (forced - 1) % N;
    const int groups = a[0].groups > 1 ? a[0].groups : 1;
    double read = 0, mb = 0;                 // what the problems read of the source, at most all of it, and write
    for (int j = 0; j < count; ++j) {
        read += (double)a[j].M * a[j].Ktot * groups * es;
        mb += (double)a[j].M * a[j].Ngemm * groups * es * 1e-6;
    }
    mb += (read < a[0].src_bytes ? read : a[0].src_bytes) * 1e-6;
    double cost[N];
    int best = 0;
    for (int i = 0; i < N; ++i) {
        long blocks = 0;
        double work = 0;
        for (int j = 0; j < count; ++j) {
            const long b = (long)ceil_div(a[j].M, tiles[i].bm) * ceil_div(a[j].Ngemm, tiles[i].bn) * groups;
            const double nk = (double)(((long)a[j].Ktot * es + PK_BYTES - 1) / PK_BYTES);
            blocks += b;
            work += (double)b * (nk * tiles[i].step + tiles[i].rest);
        }
        // 256 CUs: whole rounds of the average block
        const double rounds = (double)((blocks + 255) / 256) * (work / (double)blocks), bytes = mb * tiles[i].per_mb;
        cost[i] = tiles[i].fixed + (rounds > bytes ? rounds : bytes);
        if (cost[i] < cost[best]) best = i;
    }
    // At most four k-tiles: three stages of 256 x 128, one block a CU, leave the loads of a block exposed in front of its stores.  Two stages of
    // 128 x 128 let two blocks share a CU, one loading while the other stores, once there are more than two rounds of the larger blocks
    // (us, larger / these, with statistics: 256 -> 1024 1x1 on 25 k pixels 36.8 / 34.3, 192 -> 768 on 40 k 38.7 / 35.4, 128 -> 512 on 100 k
    // 50.8 / 47.6; 256 -> 512 on 25 k, 392 blocks, 20.7 / 20.1, without statistics 19.2 / 19.5; eight k-tiles, 512 -> 2048 on 6 k, 25.3 / 27.2).
    auto short_reduction = [&](int i) {
        return es == 2 && i == 0 && a[0].Ktot * 2 <= 4 * PK_BYTES && block_count(tiles[0], a, count) > 512 ? kShort : i;
    };
    if (es != 2 || !stats || tiles[best].wk > 1) return short_reduction(best);   // (fp32: no shape gained)
    for (int i = 0; i < N; ++i) cost[i] += tiles[i].stats + 1.5e-3 * ceil_div(a[0].M, tiles[i].bm) * tiles[i].rows;
    for (int i = 0; i < N; ++i)
        if (tiles[i].wk == 1 && cost[i] < cost[best]) best = i;
    return short_reduction(best);
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int ST, int NP, bool GATHER> int launch_np(const IgemmArgs *a, int count, hipStream_t stream)
{
    PipeProblems<NP> pp;
    int most = 0;
    pp.tiles_n = ceil_div(a[0].Ngemm, BN);
    for (int j = 0; j < count; ++j) {
        pp.a[j] = a[j];
        pp.tiles_m[j] = ceil_div(a[j].M, BM);
        pp.cols[j] = a[j].wpk_bytes > a[j].src_bytes && a[j].src_bytes <= (4u << 20) && pp.tiles_n >= 8;
        pp.by[j] = make_div(pp.cols[j] ? pp.tiles_m[j] : pp.tiles_n);
        if (pp.tiles_m[j] > most) most = pp.tiles_m[j];
    }
    hipLaunchKernelGGL((igemm_pipe_kernel<T, BM, BN, WM, WN, WK, ST, NP, GATHER>), dim3((unsigned)most * pp.tiles_n, count, a[0].groups),
                       dim3(64 * WM * WN * WK), 0, stream, pp);
    return check_launch();
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int ST, bool GATHER = false> int launch(const IgemmArgs *a, int count, hipStream_t stream)
{
    return count == 1 ? launch_np<T, BM, BN, WM, WN, WK, ST, 1, GATHER>(a, 1, stream)
                      : launch_np<T, BM, BN, WM, WN, WK, ST, kMaxProblems, GATHER>(a, count, stream);
}

}  // namespace

// One problem, or the residue classes of one strided backward-data pass (same tensors, filters of their own; a class that no
// tap reaches has ntaps = 0 and is filled with zeros).  groups, src_ld and vec_out are set; the caller has checked that
// channel runs are 16-byte granular.
int launch_igemm_pipe(int dtype, const IgemmArgs *a, int count, hipStream_t stream)
{
    if (count < 1 || count > kMaxProblems) return NSK_ERR_BAD_DESC;
    if (dtype == NSK_BF16) {
        switch (cheapest(kTilesBf16, 2, a, count, a->stats != nullptr)) {
        case 0: return launch<bf16_t, 256, 128, 4, 2, 1, 3>(a, count, stream);
        case 1: return launch<bf16_t, 128, 128, 2, 4, 1, 4>(a, count, stream);
        case 2: return launch<bf16_t, 256, 64, 4, 2, 1, 3>(a, count, stream);
        case 3:   // (four stages where a CU gets one block: 512 -> 512 3x3 at 14x14, N=16 28.9 -> 27.3 us)
            return block_count(kTilesBf16[3], a, count) > 256 ? launch<bf16_t, 128, 64, 4, 2, 1, 3>(a, count, stream)
                                                             : launch<bf16_t, 128, 64, 4, 2, 1, 4>(a, count, stream);
        case 4: return launch<bf16_t, 64, 64, 2, 2, 2, 3>(a, count, stream);
        case kShort: return launch<bf16_t, 128, 128, 2, 4, 1, 2>(a, count, stream);
        default: return launch<bf16_t, 128, 32, 4, 1, 1, 3>(a, count, stream);
        }
    }
    if (a->gather) return launch<float, 32, 32, 1, 1, 4, 4, true>(a, count, stream);
    switch (cheapest(kTilesF32, 4, a, count, a->stats != nullptr)) {
    case 0: return launch<float, 128, 64, 2, 1, 2, 3>(a, count, stream);
    case 1: return launch<float, 64, 64, 1, 2, 2, 3>(a, count, stream);
    case 2: return launch<float, 256, 128, 4, 2, 1, 3>(a, count, stream);
    case 3: return launch<float, 128, 32, 4, 1, 1, 3>(a, count, stream);
    case 4: return launch<float, 64, 32, 2, 1, 2, 4>(a, count, stream);
    default: return launch<float, 32, 32, 1, 1, 4, 4>(a, count, stream);
    }
}

// The packing of a small filter is a launch (2.5 us, and as much on the host) for next to no work; fetched four bytes a lane, a k-tile of
// the smallest shape takes 0.2 us more.  Up to eight k-tiles, us, packed / fetched, in a graph: 16 -> 16 3x3 at 32x32 N=8 8.1 / 7.2, 64 -> 64 1x1
// at 56x56 6.7 / 5.3, 128 -> 128 1x1 stride 2 7.6 / 6.4, 256 -> 128 1x1 (eight) 8.1 / 8.3; 64 -> 64 3x3 (18) 10.5 / 13.1.  Launched one
// by one, all three passes of the first 27.0 / 20.6.
bool igemm_pipe_gathers(int dtype, const IgemmArgs *a, int count)
{
    if (dtype != NSK_F32 || count < 1 || count > kMaxProblems || a->groups > 1) return false;
    for (int j = 0; j < count; ++j)
        if (a[j].Ktot > 8 * PK_BYTES / 4) return false;
    return cheapest(kTilesF32, 4, a, count, false) == kSmallest;
}

int igemm_pipe_stats_rows(int dtype, const IgemmArgs &a)
{
    const PipeTile &t = dtype == NSK_BF16 ? kTilesBf16[cheapest(kTilesBf16, 2, &a, 1, true)] : kTilesF32[cheapest(kTilesF32, 4, &a, 1, true)];
    return ceil_div(a.M, t.bm) * t.rows;
}

}  // namespace nsk
