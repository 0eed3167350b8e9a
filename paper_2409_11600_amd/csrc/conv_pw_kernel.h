// Kernel template of the short-reduction convolution (see conv_pw.hip for the description); included by the
// translation units that instantiate it (64-channel output chunks in conv_pw.hip, 16- and 32-channel outputs in
// conv_pw_narrow16.hip and conv_pw_narrow32.hip), so that they compile side by side.
#pragma once
#include <stdlib.h>

#include "nsk_internal.h"

namespace nsk {

struct PwArgs {
    IgemmArgs g;
    int tiles;
    int zero_cell;   // also write zeros to the other pixels of each row's 2x2 output cell (see IgemmArgs::zero_cell)
    // Wide outputs whose filter does not fit in LDS are split into col_groups column groups of `cols` channels: a block
    // keeps one group's filter and walks over the tiles of its share of the rows (col_groups divides 32; 1 = no split).
    int cols, col_groups;
    unsigned out_bytes;
    unsigned long long magic_img, magic_row;   // ceil(2^40 / (Mi*Mj)), ceil(2^40 / Mj)
};
// outputs of 16 and of 32 channels (instantiated in conv_pw_narrow16.hip / conv_pw_narrow32.hip); NSK_ERR_UNSUPPORTED for
// a shape without an instance
int launch_conv_pw_narrow16(const PwArgs &pa, hipStream_t stream);
int launch_conv_pw_narrow32(const PwArgs &pa, hipStream_t stream);
// (k-steps, taps) pairs the narrow translation units instantiate
inline bool conv_pw_narrow_instance(int ks, int taps)
{
    const int kpt = taps > 0 && ks % taps == 0 ? ks / taps : 0;     // 16-channel steps per tap
    if (!(taps == 1 || taps == 2 || taps == 4 || taps == 9)) return false;
    return kpt == 1 || kpt == 2 || (kpt == 4 && taps != 9);
}

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPwGrid = 256;            // blocks (see pw_grid); a shape property, as the number of statistics rows is
constexpr unsigned PW_OOB = 0xF0000000u;  // beyond every buffer: loads return zero, stores are dropped
constexpr int PW_MAX_NCH = 4;           // column chunks of 64 (Ngemm <= 256)

constexpr int pw_blocks_per_cu(int taps, int nw) { return nw < 64 && taps == 9 ? 2 : 1; }   // (the registers they may have)

template <int KS, int FM, int TAPS, bool ACC, int NW>
__global__ __launch_bounds__(256, pw_blocks_per_cu(TAPS, NW)) void conv_pw_kernel(const PwArgs pa)
{
    const IgemmArgs &a = pa.g;
    constexpr int NCH = NW == 64 ? PW_MAX_NCH : 1;   // chunks
    constexpr int TM = 32 * FM;                      // pixels per wavefront tile
    constexpr int RPL = (TM + 63) / 64;              // tile rows decoded per lane
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int KPT = KS / TAPS;                   // k-steps (16 channels) per tap
    // Output channels are handled in chunks of NW (64, or the whole of a 32- or 16-channel output).
    constexpr int FN = NW == 64 ? 2 : 1;             // 32-channel MFMA tiles per chunk
    constexpr int SROW = NW * 2 + 16;                // staged bytes per pixel: NW channels and a 16-byte pad
    constexpr int SROW_F32 = NW * 4 + 16;            // the same for fp32 sums (accumulating launches)
    constexpr int CPP = NW / 8;                      // 16-byte pieces of a pixel's chunk
    constexpr int JJ = 32 * CPP / 64 > 0 ? 32 * CPP / 64 : 1;   // pieces per lane and 32-pixel fragment
    constexpr int STRIP = ACC ? 32 * SROW_F32 : 32 * SROW;      // bytes of the transposing strip
    const int Cs = 16 * KPT;
    const int WROW = KS * 32 + 16;                   // filter row pitch: 16 bytes of padding spread the rows over the banks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int frow = lane & 31, fk = lane >> 5;
    unsigned char *w_lds = smem;
    const int w_rows = pa.cols < 32 ? 32 : pa.cols;   // filter rows in LDS (a 16-channel output still multiplies 32: the rest are zero)
    unsigned char *my_st = smem + (size_t)w_rows * WROW + wave * (STRIP + (2 * TAPS + 2) * TM * 4);
    unsigned *soff_lds = (unsigned *)(my_st + STRIP);   // [2][TAPS][TM] byte offsets of the tile's source pixels
    unsigned *ooff_lds = soff_lds + 2 * TAPS * TM;             // [2][TM] byte offsets of its output pixels (+ flags)

    const __amdgpu_buffer_rsrc_t src_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.src, 0, a.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wpk_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.wpk, 0, a.wpk_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t out_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, pa.out_bytes, 0x00020000);

    // filter -> LDS
    // block id -> (column group, row share).  Consecutive ids go to different XCDs, so the column groups of one row
    // share get ids that differ by a multiple of 8: they read the same pixels through one XCD's L2.
    const int cg = ((int)blockIdx.x >> 3) % pa.col_groups;
    const int rb = ((int)blockIdx.x & 7) + 8 * (((int)blockIdx.x >> 3) / pa.col_groups);
    const int n_rb = (int)gridDim.x / pa.col_groups;      // row shares
    const int col0 = cg * pa.cols;                        // first output channel of this block
    // Wide filters, and 32 channels x nine taps just packed by the launch before (backward-data): the first pieces are requested here and
    // stored behind the request of the first tile, so that a block waits for memory once (64 -> 256 1x1, 64 images of 56x56, 31.1 ->
    // 30.1 us; backward-data of 16 -> 32 3x3, 128 and 256 images of 32x32, 12.5 -> 12.1, 18.8 -> 17.7; 32 -> 32 3x3, 64 images of 16x16, 7.5 ->
    // 7.0).  With small filters, and with those that lie in the caches from the pass before, that order is slower: 64 -> 32 1x1, 256
    // images of 32x32, 11.4 -> 12.2; forward 16 -> 32 3x3 stride 2, 256 images of 32x32, 6.3 -> 6.8; 16 -> 16 3x3, 64 images, 4.4 -> 4.9;
    // 32 -> 32 3x3 stride 2, 128 images, 7.2 -> 7.5.
    constexpr bool MAY_EARLY = (TAPS == 9 && KS == 18) || (NW == 64 && KS >= 4);
    const bool early = MAY_EARLY && (TAPS != 9 || a.packed);
    constexpr int FL = 6;
    const int pieces = w_rows * (2 * KS);
    u32x4 fv[FL];
    auto filter_at = [&](int idx) -> u32x4 {
        const int n = idx / (2 * KS), ch = idx % (2 * KS);
        return __builtin_amdgcn_raw_buffer_load_b128(wpk_rsrc, n < pa.cols ? (unsigned)(((col0 + n) * KS * 16 + ch * 8) * 2) : PW_OOB, 0, 0);
    };
    auto filter_to_lds = [&](int idx, u32x4 v) {
        if (idx < pieces) *(u32x4 *)(w_lds + idx / (2 * KS) * WROW + idx % (2 * KS) * 16) = v;
    };
    if (early) {
#pragma unroll
        for (int i = 0; i < FL; ++i) fv[i] = filter_at(tid + 256 * i);
    } else {
        for (int idx = tid; idx < pieces; idx += 256) filter_to_lds(idx, filter_at(idx));
        lds_barrier();
    }

    const int per_img = a.Mi * a.Mj;
    // Source (per tap) and output byte offsets of the tile's pixels (PW_OOB for rows past the end and for source
    // positions outside the image), written to this wavefront's LDS arrays of the given parity.  Output offsets are
    // multiples of 16; their two low bits say whether the pixel to the right / below exists (zero_cell).
    auto decode = [&](int tile, int par) {
#pragma unroll
        for (int u = 0; u < RPL; ++u) {
            const int r = lane + 64 * u;
            const int m = tile * TM + r;
            unsigned so[TAPS], oo = PW_OOB;
#pragma unroll
            for (int tp = 0; tp < TAPS; ++tp) so[tp] = PW_OOB;
            if (r < TM && m < a.M) {
                const int img = (int)(((unsigned long long)m * pa.magic_img) >> 40);
                const int rem = m - img * per_img;
                const int i = (int)(((unsigned long long)rem * pa.magic_row) >> 40);
                const int j = rem - i * a.Mj;
#pragma unroll
                for (int tp = 0; tp < TAPS; ++tp) {
                    const int h = i * a.mult_h + a.add_h + a.off_h[tp], w = j * a.mult_w + a.add_w + a.off_w[tp];
                    if ((unsigned)h < (unsigned)a.Hs && (unsigned)w < (unsigned)a.Ws)
                        so[tp] = (unsigned)(((img * a.Hs + h) * a.Ws + w) * Cs) * 2u;
                }
                const int ho = i * a.osh + a.oa, wo = j * a.osw + a.ob;
                oo = (unsigned)(((img * a.Ho + ho) * a.Wo + wo) * a.Co) * 2u;
                oo |= (wo + 1 < a.Wo ? 1u : 0u) | (ho + 1 < a.Ho ? 2u : 0u);
            }
            if (r < TM) {
#pragma unroll
                for (int tp = 0; tp < TAPS; ++tp) soff_lds[(par * TAPS + tp) * TM + r] = so[tp];
                ooff_lds[par * TM + r] = oo;
            }
        }
    };
    auto issue = [&](u32x4 (&A)[FM][KS], int par) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
#pragma unroll
            for (int tp = 0; tp < TAPS; ++tp) {
                const unsigned so = soff_lds[(par * TAPS + tp) * TM + 32 * mi + frow] + (unsigned)(fk * 16);
#pragma unroll
                for (int kk = 0; kk < KPT; ++kk)
                    A[mi][tp * KPT + kk] = __builtin_amdgcn_raw_buffer_load_b128(src_rsrc, so + kk * 32, 0, 0);
            }
        }
    };

    // Accumulating launches: the old values of the 64-channel chunk a lane will store (same pixel, same 16 bytes),
    // fetched one chunk ahead of the multiply that needs them.
    u32x4 O[2][FM][JJ];
    auto issue_old = [&](u32x4 (&Ob)[FM][JJ], int par, int nc) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int jj = 0; jj < JJ; ++jj) {
                const int idx = lane + 64 * jj, pos = idx / CPP, ck = idx % CPP;
                const unsigned oo = ooff_lds[par * TM + 32 * mi + pos] & ~15u;
                Ob[mi][jj] = __builtin_amdgcn_raw_buffer_load_b128(out_rsrc, oo + (unsigned)((col0 + nc * NW + ck * 8) * 2), 0, 0);
            }
    };

    float ssum[NCH][8], ssq[NCH][8];
#pragma unroll
    for (int nc = 0; nc < NCH; ++nc)
#pragma unroll
        for (int e = 0; e < 8; ++e) ssum[nc][e] = ssq[nc][e] = 0.f;
    const int nch = pa.cols / NW;
    const bool want_stats = a.stats != nullptr;

    auto compute = [&](const u32x4 (&A)[FM][KS], int par, bool has_next) {
#pragma unroll
        for (int nc = 0; nc < NCH; ++nc) {
            if (nc >= nch) break;
            if constexpr (ACC) {
                if (nc + 1 < nch) issue_old(O[(nc + 1) & 1], par, nc + 1);
            }
            f32x16 acc[FM][FN];
#pragma unroll
            for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
            const unsigned char *wb = w_lds + (nc * NW + frow) * WROW + fk * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 bfr[FN];
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) bfr[ni] = *(const bf16x8 *)(wb + ni * 32 * WROW + ks * 32);
#pragma unroll
                for (int mi = 0; mi < FM; ++mi) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, A[mi][ks]);
#pragma unroll
                    for (int ni = 0; ni < FN; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ni], av, acc[mi][ni], 0, 0, 0);
                }
            }
            // acc[mi][ni][4g+j] = channel NW*nc + 32ni + 8g + 4fk + j of pixel 32mi + frow: round, transpose 32 pixels x NW
            // channels through the strip, store the chunk of a pixel (128, 64 or 32 bytes) with CPP lanes.
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) {
#pragma unroll
                for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        if (ni * 32 + g * 8 >= NW) continue;      // a 16-channel output uses half of the MFMA tile
                        if constexpr (ACC) {
                            *(f32x4 *)(my_st + frow * SROW_F32 + (ni * 32 + g * 8 + fk * 4) * 4) =
                                f32x4{acc[mi][ni][g * 4], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]};
                        } else {
                            bf16x4 pk;
#pragma unroll
                            for (int j = 0; j < 4; ++j) pk[j] = (bf16_t)acc[mi][ni][g * 4 + j];
                            *(bf16x4 *)(my_st + frow * SROW + (ni * 32 + g * 8 + fk * 4) * 2) = pk;
                        }
                    }
#pragma unroll
                for (int jj = 0; jj < JJ; ++jj) {
                    const int idx = lane + 64 * jj, pos = idx / CPP, ck = idx % CPP;
                    u32x4 v;
                    if constexpr (ACC) {
                        // old value + sum of products, rounded to the storage type once
                        const f32x4 lo = *(const f32x4 *)(my_st + pos * SROW_F32 + ck * 32);
                        const f32x4 hi = *(const f32x4 *)(my_st + pos * SROW_F32 + ck * 32 + 16);
                        const bf16x8 old = __builtin_bit_cast(bf16x8, O[nc & 1][mi][jj]);
                        bf16x8 r;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            r[e] = (bf16_t)(lo[e] + (float)old[e]);
                            r[e + 4] = (bf16_t)(hi[e] + (float)old[e + 4]);
                        }
                        v = __builtin_bit_cast(u32x4, r);
                    } else {
                        v = *(const u32x4 *)(my_st + pos * SROW + ck * 16);
                    }
                    const unsigned oraw = ooff_lds[par * TM + 32 * mi + pos];
                    const unsigned oo = oraw & ~15u, cb = (unsigned)((col0 + nc * NW + ck * 8) * 2);
                    __builtin_amdgcn_raw_buffer_store_b128(v, out_rsrc, oo + cb, 0, 0);
                    if (!ACC && pa.zero_cell) {
                        const u32x4 z = {0u, 0u, 0u, 0u};
                        const unsigned right = (unsigned)(a.Co * 2), below = (unsigned)(a.Wo * a.Co * 2);
                        __builtin_amdgcn_raw_buffer_store_b128(z, out_rsrc, (oraw & 1u) ? oo + right + cb : PW_OOB, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b128(z, out_rsrc, (oraw & 2u) ? oo + below + cb : PW_OOB, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b128(z, out_rsrc, (oraw & 3u) == 3u ? oo + below + right + cb : PW_OOB, 0, 0);
                    }
                    if (!ACC && want_stats && oo != PW_OOB) {
                        const bf16x8 bv = __builtin_bit_cast(bf16x8, v);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float f = (float)bv[e];
                            ssum[nc][e] += f;
                            ssq[nc][e] += f * f;
                        }
                    }
                }
            }
        }
        if constexpr (ACC) {
            if (has_next) issue_old(O[0], par ^ 1, 0);   // first chunk of the next tile (its offsets are decoded already)
        }
    };

    u32x4 A0[FM][KS], A1[FM][KS];
    const int stride = n_rb * 4;
    // few tiles: spread them over the CUs first (one wavefront per CU) instead of filling the first blocks
    int t = pa.tiles >= stride ? rb * 4 + wave : wave * n_rb + rb;
    if (t < pa.tiles) {
        decode(t, 0);
        if constexpr (ACC) issue_old(O[0], 0, 0);
        issue(A0, 0);
    }
    if (early) {
        for (int at = tid;;) {
#pragma unroll
            for (int i = 0; i < FL; ++i) filter_to_lds(at + 256 * i, fv[i]);
            at += 256 * FL;
            if (at - tid >= pieces) break;
#pragma unroll
            for (int i = 0; i < FL; ++i) fv[i] = filter_at(at + 256 * i);
        }
        lds_barrier();
    }
    while (t < pa.tiles) {
        bool has_next = t + stride < pa.tiles;
        if (has_next) {
            decode(t + stride, 1);
            issue(A1, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute(A0, 0, has_next);
        __builtin_amdgcn_sched_barrier(0);
        t += stride;
        if (t >= pa.tiles) break;
        has_next = t + stride < pa.tiles;
        if (has_next) {
            decode(t + stride, 0);
            issue(A0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute(A1, 1, has_next);
        __builtin_amdgcn_sched_barrier(0);
        t += stride;
    }

    if (!ACC && want_stats) {
        // lanes with equal (lane % CPP) hold the same channels: add them up; then the wavefronts' sums through their strips, in
        // order: one row of partial sums per block where it has all columns
        float *const mine = (float *)my_st;              // [2][cols]
#pragma unroll
        for (int nc = 0; nc < NCH; ++nc) {
            if (nc >= nch) break;
            store_folded<CPP>(ssum[nc], ssq[nc], mine + nc * NW, (size_t)pa.cols);
        }
        lds_barrier();
        const int pitch = (STRIP + (2 * TAPS + 2) * TM * 4) / 4;
        const float *first = (const float *)(smem + (size_t)w_rows * WROW);
        for (int c = tid; c < 2 * pa.cols; c += 256) {
            const int which = c >= pa.cols;
            float *to = a.stats + (size_t)which * a.stats_rows * a.Ngemm + col0 + c - which * pa.cols;
            if (pa.col_groups > 1) {       // (few row shares: a row per wavefront)
#pragma unroll
                for (int w = 0; w < 4; ++w) to[(size_t)(4 * rb + w) * a.Ngemm] = first[c + w * pitch];
            } else {
                // (in fp64, rounded once: sums in fp32 go no further than a wavefront's own pixels)
                to[(size_t)rb * a.Ngemm] = (float)(((double)first[c] + (double)first[c + pitch]) + ((double)first[c + 2 * pitch] + (double)first[c + 3 * pitch]));
            }
        }
    }
}

inline int pw_chunk(const IgemmArgs &a) { return a.Ngemm % 64 == 0 ? 64 : a.Ngemm; }   // NW: 64, 32 or 16

// Output channels per block: all of them if their filter fits in LDS, else the largest multiple of 64 that does and
// splits the columns into 2, 4, ... 32 groups; 0 if there is none.
inline int pw_cols(const IgemmArgs &a)
{
    const long limit = a.ntaps == 9 ? 36864 : 32768;       // filter elements a block keeps in LDS
    if (a.Ngemm <= 64 * PW_MAX_NCH && (long)a.Ngemm * a.Ktot <= limit) return a.Ngemm;
    if (a.Ngemm % 64 != 0) return 0;
    for (int cols = 64 * PW_MAX_NCH; cols >= 64; cols -= 64) {
        if ((long)cols * a.Ktot > limit || a.Ngemm % cols != 0) continue;
        const int groups = a.Ngemm / cols;
        if (groups <= 32 && 32 % groups == 0) return cols;
    }
    return 0;
}

inline int pw_tile_rows(const IgemmArgs &a) { return a.Ngemm <= 32 && a.ntaps == 9 && a.Ktot == 288 ? 32 : 64; }

inline size_t pw_smem(const IgemmArgs &a, int tm)
{
    const int nw = pw_chunk(a), cols = pw_cols(a);
    return (size_t)(cols < 32 ? 32 : cols) * (a.Ktot * 2 + 16) +
           4 * (size_t)(32 * (a.accumulate ? nw * 4 + 16 : nw * 2 + 16) + (2 * a.ntaps + 2) * tm * 4);
}

// Blocks of a launch: one a CU, or two, where registers and LDS allow it, as four wavefronts a CU leave part of the load, multiply and
// store phases of a tile exposed:
//   * 3x3 filters of narrow outputs, while every wavefront then still has a tile.  us, one / two: 16 -> 16 256 images
//     of 32x32 10.4 / 8.9, 128 of 56x56 14.6 / 11.5 (four blocks of 32-pixel tiles 11.2, but 14.4 with statistics against 13.4),
//     32 -> 32 64 of 56x56 17.4 / 13.6;
//   * one tap of at most 64 channels, from one tile per wavefront of the smaller grid.  us, one / two, with statistics, 56x56: 64 -> 64 21
//     images 9.0 / 8.1, 64 images 16.3 / 14.3; 64 -> 256 64 images 42.9 / 33.5, 128 images 66.5 / 58.8; 32 -> 64 128 images
//     19.6 / 15.5.  Operands beyond 300 MB stream better to one block a CU (64 -> 64 410 MB 76.3 / 77.4, 64 -> 128 617 MB 120 / 126), as do
//     128 channels (128 -> 64 128 images 36.7 / 40.1).
inline int pw_grid(const IgemmArgs &a)
{
    if (a.Ngemm <= 32) return a.ntaps == 9 && ceil_div(a.M, pw_tile_rows(a)) >= 2 * kPwGrid * 4 ? 2 * kPwGrid : kPwGrid;
    const bool streams = (long)a.Nimg * a.Ho * a.Wo * a.Co * 2 + (long)a.src_bytes > 300000000L;
    return a.ntaps == 1 && a.Ktot <= 64 && pw_cols(a) == a.Ngemm && ceil_div(a.M, 64) >= kPwGrid * 4 && !streams ? 2 * kPwGrid : kPwGrid;
}

template <int KS, int FM, int TAPS, bool ACC, int NW> int launch_pw_acc(PwArgs pa, hipStream_t stream)
{
    pa.tiles = ceil_div(pa.g.M, 32 * FM);
    pa.cols = pw_cols(pa.g);
    pa.col_groups = pa.g.Ngemm / pa.cols;
    // at least half of a CU's LDS, so that 256 blocks land on 256 different CUs
    size_t smem = pw_smem(pa.g, 32 * FM);
    if (pw_grid(pa.g) == kPwGrid && smem < 84 * 1024) smem = 84 * 1024;
    const int rc = allow_lds<conv_pw_kernel<KS, FM, TAPS, ACC, NW>>(160 * 1024);
    if (rc != NSK_OK) return rc;
    hipLaunchKernelGGL((conv_pw_kernel<KS, FM, TAPS, ACC, NW>), dim3(pw_grid(pa.g)), dim3(256), smem, stream, pa);
    return check_launch();
}

template <int KS, int FM, int TAPS, int NW> int launch_pw(const PwArgs &pa, hipStream_t stream)
{
    return pa.g.accumulate ? launch_pw_acc<KS, FM, TAPS, true, NW>(pa, stream)
                           : launch_pw_acc<KS, FM, TAPS, false, NW>(pa, stream);
}

}  // namespace
}  // namespace nsk
