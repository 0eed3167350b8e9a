// Backward-weight convolution for every layer without a kernel of its own whose channel runs are 16-byte granular (fp32
// and bf16, grouped launches): the pipelined split-K kernel.
//
//   part[split][k][tap][c] = sum over the split's output pixels l of dy[l][k] * x[pixel(l) shifted by tap][c]
//
// GEMM view: rows = output channels k, columns n = (tap, input channel), reduction over the output pixels, split across
// blocks into float partial sums that a second kernel adds in a fixed order (bitwise reproducible, no atomics).
//
// What bounds it: both operands lie with the reduction index as the slow one.  The kernel before this one transposed bf16
// tiles with 2-byte LDS writes and had one k-tile of 32 pixels in flight: 512 -> 512 channels, 3x3 at 7x7, N=64 took 54 us
// where the matrix units need 8.  Here k-tiles of KT pixels go from memory straight into LDS exactly as they lie there
// ([pixel][channel], 16 bytes per lane, no registers), ST deep, with one counted wait and one barrier each; bf16 fragments
// come out through the transposing LDS read (8 consecutive pixels of one channel per lane), fp32 ones as 4-byte reads.
//
// LDS: unpadded pixel rows (a direct load writes 1 KB in one piece).  The 16 rows x 64 bytes (bf16: 4 rows x 64 bytes
// per clock) or two rows x 128 bytes (fp32) that one fragment read serves at once would fall into the same banks, so a
// row's 64-byte (fp32: 128-byte) pieces are exchanged with its number; the exchange is made in the source address.
//
// Sums: the products of ST k-tiles are added up in one or two sets of accumulators (alternately) and those then added to another,
// so that the error does not grow with the length of a split.  Short splits, up to kLong k-tiles, have two sets: chains of
// 64 pixels in fp32, 8 products of 16 pixels in bf16.  Long ones, whose error was larger before, have twice as long chains:
// eight k-tiles in two sets (fp32), one set (bf16), where the adds would take 3%.  Error against 64 bits (2-norm,
// random data; one set, 16-18 k-tiles / this / the kernels before): fp32 16->16 at 32x32 N=8 2.15e-7, 1.61e-7, 1.61e-7;
// 744->744 1x1 stride 2 at 24x24 N=3 3.73e-7, 1.48e-7, 1.63e-7; 128->128 at 28x28 N=64 4.06e-7, 2.30e-7, 4.99e-7; bf16
// 416->416 1x1 at 25x25 N=3 1.14e-7, 0.77e-7, 0.81e-7; 512->512 at 7x7 N=64 1.75e-7, 1.07e-7, 1.52e-7.  Time
// up to 3% more in fp32, 1-3% less in bf16.
//
// fp32 from about 1 GFLOP on: products of bf16 pieces (nsk_internal.h), 64 x 64 outputs a wavefront so that each piece is used twice, the
// k-tile's two groups of 16 pixels to a pair of wavefronts whose sums meet in LDS at the end.  Bound by the vector unit (208 instructions
// for the pieces and about 80 of addresses for 24 products of 32 clocks).  One chain for the large products and one for the small, no
// banking (a third set of sums does not fit in the registers of two wavefronts a SIMD), so splits are at most kPieces k-tiles.  Fp32 unit /
// this, us with the reduction, and error: 128->128 3x3 at 28x28 N=64 140 / 103, 2.2e-7 / 1.8e-7; 256->256 at 14x14 N=32 78 / 57, 2.0e-7 /
// 1.3e-7; 72->100 at 29x37 N=20 44 / 38, 2.0e-7 / 1.2e-7; 64->64 at 32x32 N=128 96 / 86, 2.2e-7 / 1.8e-7.
#include "nsk_internal.h"

namespace nsk {
namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr int kLong = 16;     // see Sums
constexpr int kPieces = 64;   // most k-tiles of a split on bf16 pieces, see Sums

struct PipeArgs {
    WgradArgs g;
    Div by_pq, by_q;
    int tiles_n, tiles_k;
    unsigned x_bytes, dy_bytes;
};

// exchange of 16-byte pieces inside pixel row r (row bytes RB): see above
template <int ES, int RB> __device__ constexpr int piece_swap(int r)
{
    if constexpr (ES == 4) return (r & 1) << 3;
    else if constexpr (RB == 256) return (r & 3) << 2;
    else return ((r >> 1) & 1) << 2;
}

// WK = 2 (fp32): products of bf16 pieces, every other 16 pixels of a k-tile by each wavefront of a pair, whose sums are added at the end.
template <typename T, int BM, int BN, int WM, int WN, int WK, int KT, int ST, int CH>
__global__ __launch_bounds__(64 * WM * WN * WK, WK == 2 ? 2 : 1) void wgrad_pipe_kernel(const PipeArgs w)
{
    const WgradArgs &a = w.g;
    constexpr int ES = (int)sizeof(T), VEC = 16 / ES, NW = WM * WN * WK;
    constexpr bool SPLIT = WK == 2;
    static_assert(!SPLIT || (ES == 4 && KT == 32 && ST == 3 && CH == 1), "two groups of 16 pixels");
    constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    constexpr int RBA = BM * ES, RBX = BN * ES;                 // bytes of a pixel row
    constexpr int PA = RBA / 16, PX = RBX / 16;                 // its 16-byte pieces
    constexpr int ROWS_A = 64 / PA, ROWS_X = 64 / PX;           // pixel rows of one direct load
    constexpr int LA = KT / ROWS_A / NW, LX = KT / ROWS_X / NW; // direct loads per wavefront and k-tile
    static_assert(LA >= 1 && LX >= 1 && LA * ROWS_A * NW == KT && LX * ROWS_X * NW == KT, "whole loads");
    static_assert(ES == 2 ? (RBA == 128 || RBA == 256) && (RBX == 128 || RBX == 256) : RBA % 256 == 0 && RBX % 256 == 0, "row exchange");
    static_assert(ST == 3 || ST == 4, "stages");
    // one variable per stage and operand: the compiler keeps the reads of one apart from the direct loads into the others
    __shared__ __attribute__((aligned(1024))) unsigned char sa0[KT * RBA], sa1[KT * RBA], sa2[KT * RBA], sa3[ST == 4 ? KT * RBA : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char sx0[KT * RBX], sx1[KT * RBX], sx2[KT * RBX], sx3[ST == 4 ? KT * RBX : 16];
#define NSK_STAGE(S, P) ((S) == 0 ? P##0 : (S) == 1 ? P##1 : (S) == 2 ? P##2 : P##3)

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wk = wave % WK, wm = wave / WK / WN, wn = wave / WK % WN;
    const int frow = lane & 31, fk = lane >> 5;
    // grouped convolution: blockIdx.z names the group.  Tiles of one split next to each other on one XCD (blocks go to the
    // eight XCDs in turn), whose L2 then holds the pixel rows they share.
    const int grp = blockIdx.z, tiles = w.tiles_n * w.tiles_k;
    int split, tile;
    {
        const int total = tiles * a.splits, x = blockIdx.x & 7, i = blockIdx.x >> 3;
        const int q = total >> 3, r = total & 7;
        const int t = x * q + min(x, r) + i;
        split = t / tiles;
        tile = t - split * tiles;
    }
    const int tk = tile / w.tiles_n, tn = tile - tk * w.tiles_n;
    const int n0 = tn * BN, k0 = tk * BM, NT = a.ntaps * a.C;
    const int l_begin = split * a.rows_per_split, l_end = min(a.L, l_begin + a.rows_per_split);
    const int nk = (l_end - l_begin + KT - 1) / KT;

    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, w.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t dy_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.dy, 0, w.dy_bytes, 0x00020000);

    // This lane's columns: fixed pieces of its pixel rows, so a fixed channel of dy and a fixed (tap, channel) of x.
    // Offsets are made out of range (zeros) with bit operations: a branch around a direct load would split it in two.
    const int ra = lane / PA, rx = lane / PX;
    const int ka = k0 + ((lane % PA) ^ piece_swap<ES, RBA>(ra)) * VEC;
    const unsigned a_bad = ka < a.K ? 0u : ~0u;
    unsigned a_off[LA];
    int la, lx;                                        // pixel of this lane's first dy row, x row of the next k-tile
    const unsigned a_step = (unsigned)(KT * a.ldy * ES);
    const int nx = n0 + ((lane % PX) ^ piece_swap<ES, RBX>(rx)) * VEC;
    const unsigned x_bad = nx < NT ? 0u : ~0u;
    const int tap = nx < NT ? nx / a.C : 0;
    const int oh = a.off_h[tap] - a.ph, ow = a.off_w[tap] - a.pw;
    const unsigned xc = (unsigned)(grp * a.C + nx - tap * a.C) * ES;
    auto start_requests = [&]() {
        la = l_begin + wave * ROWS_A + ra;
        lx = l_begin + wave * ROWS_X + rx;
#pragma unroll
        for (int u = 0; u < LA; ++u) a_off[u] = (unsigned)((la + u * NW * ROWS_A) * (long)a.ldy + grp * a.K + ka) * ES;
    };
    auto request = [&](auto S) {
        constexpr int I = S.value;
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            const unsigned past = ~(unsigned)((la + u * NW * ROWS_A - l_end) >> 31);    // all ones from l_end on
            __builtin_amdgcn_raw_ptr_buffer_load_lds(dy_rsrc, (lds_void *)&NSK_STAGE(I, sa)[(wave + NW * u) * 1024], 16,
                                                     (int)(a_off[u] | a_bad | past), 0, 0, 0);
            a_off[u] += a_step;
        }
        la += KT;
#pragma unroll
        for (int u = 0; u < LX; ++u) {
            const int l = lx + u * NW * ROWS_X;
            const unsigned past = ~(unsigned)((l - l_end) >> 31);
            const int img = divide(l, w.by_pq), rem = l - img * (a.P * a.Q), p = divide(rem, w.by_q), q = rem - p * a.Q;
            const int h = p * a.sh + oh, ww = q * a.sw + ow;
            // (h and ww are far below 2^31, so the sign bits tell whether they lie inside)
            const unsigned outside = (unsigned)((h | (a.H - 1 - h) | ww | (a.W - 1 - ww)) >> 31);
            const unsigned off = (unsigned)((img * a.H + h) * a.W + ww) * (unsigned)(a.ldx * ES) + xc;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void *)&NSK_STAGE(I, sx)[(wave + NW * u) * 1024], 16,
                                                     (int)(off | x_bad | past | outside), 0, 0, 0);
        }
        lx += KT;
    };

    f32x16 acc[CH][FM][FN], sum[FM][FN];   // CH chains of products, see Sums

    // Fragment addresses.  bf16, transposing read: within 16 lanes, lanes 4j..4j+3 address pixel row j (four 8-byte pieces =
    // 16 channels) and lane i receives channel i of rows 0..3; lane (channel = lane%32, half = lane/32) of an MFMA operand
    // needs pixels 8*half .. 8*half+7 of its channel: two such reads, four rows apart.
    int fa[FM], fx[FN];
    if constexpr (ES == 2) {
        const int g16 = lane >> 4, i16 = lane & 15;
        const int row = 8 * (g16 >> 1) + (i16 >> 2), inner = 32 * (g16 & 1) + 8 * (i16 & 3);
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[i] = row * RBA + (((wm * FM + i) ^ (piece_swap<ES, RBA>(row) >> 2)) * 64) + inner;
#pragma unroll
        for (int i = 0; i < FN; ++i) fx[i] = row * RBX + (((wn * FN + i) ^ (piece_swap<ES, RBX>(row) >> 2)) * 64) + inner;
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[i] = fk * RBA + (((wm * FM + i) * 32 + frow) * 4 ^ (fk << 7));
#pragma unroll
        for (int i = 0; i < FN; ++i) fx[i] = fk * RBX + (((wn * FN + i) * 32 + frow) * 4 ^ (fk << 7));
    }
    // PIECES: fp32 products of bf16 pieces
    auto multiply = [&](auto PIECES, auto S) {
        constexpr int I = S.value;
        if constexpr (decltype(PIECES)::value) {
            // lane (channel, half) holds pixels half, half + 2, ... of its group of 16, the same of both operands
            Pieces pa[FM], pb[FN];
            const int g = wk * 16;
            auto split = [&](const unsigned char *col, auto ROW) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = *(const float *)(col + (g + 2 * e) * ROW.value);
                return split3(x);
            };
#pragma unroll
            for (int i = 0; i < FM; ++i) pa[i] = split(&NSK_STAGE(I, sa)[fa[i]], std::integral_constant<int, RBA>{});
#pragma unroll
            for (int i = 0; i < FN; ++i) pb[i] = split(&NSK_STAGE(I, sx)[fx[i]], std::integral_constant<int, RBX>{});
            multiply_pieces<false>(pa, pb, acc[0], sum);
        } else if constexpr (ES == 2) {
#pragma unroll
            for (int ks = 0; ks < KT / 16; ++ks) {
                bf16x8 af[FM], bx[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&NSK_STAGE(I, sa)[fa[i] + ks * 16 * RBA]);
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&NSK_STAGE(I, sa)[fa[i] + (ks * 16 + 4) * RBA]);
                    af[i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
#pragma unroll
                for (int i = 0; i < FN; ++i) {
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&NSK_STAGE(I, sx)[fx[i] + ks * 16 * RBX]);
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)&NSK_STAGE(I, sx)[fx[i] + (ks * 16 + 4) * RBX]);
                    bx[i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
#pragma unroll
                for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < FN; ++ni)
                        acc[ks % CH][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi], bx[ni], acc[ks % CH][mi][ni], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < KT / 2 / WK; ++i) {
                const int t = wk * (KT / 2 / WK) + i;
                float af[FM], bx[FN];
#pragma unroll
                for (int m = 0; m < FM; ++m) af[m] = *(const float *)&NSK_STAGE(I, sa)[fa[m] + t * 2 * RBA];
#pragma unroll
                for (int m = 0; m < FN; ++m) bx[m] = *(const float *)&NSK_STAGE(I, sx)[fx[m] + t * 2 * RBX];
#pragma unroll
                for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < FN; ++ni)
                        acc[i % CH][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi], bx[ni], acc[i % CH][mi][ni], 0, 0, 0);
            }
        }
    };
    auto start_chains = [&]() {
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[c][mi][ni][v] = 0.f;
    };
    auto bank_sums = [&]() {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[mi][ni][v] += CH == 2 ? acc[0][mi][ni][v] + acc[CH - 1][mi][ni][v] : acc[0][mi][ni][v];
    };

    auto products = [&](auto PIECES) {
        start_requests();
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[mi][ni][v] = 0.f;
        static_for<0, ST - 1>([&](auto S) { request(S); });   // (k-tiles past the end are requested out of range: zeros)
        // The loop body is ST steps without a branch, the remainder follows: where a step could leave the loop, the compiler
        // would take the stage requested last for one that the first step reads, and wait for it.
#define NSK_STEP(S)                                                                                              \
    wait_vm<(ST - 2) * (LA + LX)>();  /* this wavefront's part of the k-tile has arrived */                      \
    __builtin_amdgcn_s_barrier();     /* everybody's has, and nobody reads the stage requested next any more */  \
    asm volatile("" ::: "memory");                                                                               \
    request(std::integral_constant<int, ((S) + ST - 1) % ST>{});                                                 \
    multiply(PIECES, std::integral_constant<int, (S)>{});
        int n = nk / ST;
        if constexpr (ES == 4 && !SPLIT) {
            static_assert(ST == 4, "eight steps are two rounds of the stages");
            for (; nk > kLong && n > 1; n -= 2) {
                start_chains();
                NSK_STEP(0)
                NSK_STEP(1)
                NSK_STEP(2)
                NSK_STEP(3)
                NSK_STEP(0)
                NSK_STEP(1)
                NSK_STEP(2)
                NSK_STEP(3)
                bank_sums();
            }
        }
        if constexpr (decltype(PIECES)::value) start_chains();   // one chain: the host keeps splits short, see kPieces
        for (; n > 0; --n) {
            if constexpr (!decltype(PIECES)::value) start_chains();
            NSK_STEP(0)
            NSK_STEP(1)
            NSK_STEP(2)
            if constexpr (ST == 4) {
                NSK_STEP(3)
            }
            if constexpr (!decltype(PIECES)::value) bank_sums();
        }
#undef NSK_STEP
        // (the last ST - 1 k-tiles have been requested; what the loop requested past the end were zeros)
#define NSK_REST(S)                             \
    wait_vm<(ST - 2 - (S)) * (LA + LX)>();      \
    __builtin_amdgcn_s_barrier();               \
    asm volatile("" ::: "memory");              \
    multiply(PIECES, std::integral_constant<int, (S)>{});
        const int rest = nk % ST;
        if constexpr (!decltype(PIECES)::value) start_chains();
        if (rest > 0) {
            NSK_REST(0)
        }
        if (rest > 1) {
            NSK_REST(1)
        }
        if constexpr (ST == 4) {
            if (rest > 2) {
                NSK_REST(2)
            }
        }
#undef NSK_REST
        wait_vm<0>();   // (nothing may still be on its way into LDS when the block gives it back)
        bank_sums();
    };
    products(std::integral_constant<bool, SPLIT>{});
    if constexpr (SPLIT) {
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[mi][ni][v] *= 1.f / kSumScale;
        if (__syncthreads_or(!finite_sums(sum))) products(std::integral_constant<bool, false>{});
        // the second wavefront of a pair hands its sums to the first, one accumulator tile at a time
        static_assert(WM * WN * 4096 <= KT * RBX, "inside a stage");
        float *red = (float *)sx0 + (wm * WN + wn) * 1024 + lane * 4;
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
                __syncthreads();
                if (wk == 1) {
#pragma unroll
                    for (int v = 0; v < 16; v += 4)
                        *(f32x4 *)(red + v * 64) = f32x4{sum[mi][ni][v], sum[mi][ni][v + 1], sum[mi][ni][v + 2], sum[mi][ni][v + 3]};
                }
                __syncthreads();
                if (wk == 0) {
#pragma unroll
                    for (int v = 0; v < 16; v += 4) {
                        const f32x4 p = *(const f32x4 *)(red + v * 64);
#pragma unroll
                        for (int j = 0; j < 4; ++j) sum[mi][ni][v + j] += p[j];
                    }
                }
            }
        if (wk == 1) return;
    }
#undef NSK_STAGE

    // sum[mi][ni][v]: row k = 32*mi + 8*(v/4) + 4*(lane/32) + v%4, column = 32*ni + lane%32 of the wavefront's sub-tile
    float *__restrict__ part = a.part + ((size_t)split * a.groups + grp) * a.K * NT;
#pragma unroll
    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
        for (int ni = 0; ni < FN; ++ni) {
            const int col = n0 + (wn * FN + ni) * 32 + frow;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = k0 + (wm * FM + mi) * 32 + 8 * (v >> 2) + 4 * fk + (v & 3);
                if (k < a.K && col < NT) part[(size_t)k * NT + col] = sum[mi][ni][v];
            }
        }
}

// Measured (us, with the reduction): bf16 3x3 512->512 at 7x7 N=64 66.8 -> 32; 3x3 stride 2 64->128 at 56x56 N=64 38.9 ->
// 21; 1x1 256->1024 at 14x14 N=128 33 -> 26 (a 256 x 128 tile with separate moving wavefronts); 3x3 16->16 at 32x32 N=256
// 21.8 -> 17; fp32 3x3 128->128 at 28x28 N=64 197 -> 150; fp32 72->100 at 29x37 N=20 65 -> 46 (39 on pieces).
//
// Tile shapes with what a k-tile, the rest of a block and the launch cost in shader clocks (bf16 measured on 35 problems, where the launch is
// left out; fp32 fitted to 260 problems of 16 to 1024 channels, 50 to 400 k pixels: 3-5% off, and the choice 0.1% off the best shape on average).
// bf16 is bound by the fill of LDS (a 128 x 128 tile brings in 32 KB per k-tile at 38 B/clk), fp32 by the matrix and vector units.
struct Shape {
    int bm, bn, kt;
    double alone, step, rest;   // clocks per k-tile where a CU has one block, and where it has several
    double fixed = 0;
    bool pieces = false;
};
constexpr Shape kBf16[] = {{128, 128, 64, 850, 850, 9000}, {64, 128, 64, 700, 700, 6000}, {64, 64, 64, 620, 450, 4000}};
constexpr Shape kF32[] = {{64, 64, 32, 1260, 1130, 2060, 5240, false}, {64, 128, 32, 1770, 1380, 4350, 7420, true}, {128, 128, 32, 2450, 2290, 12600, 790, true}};

int shapes(int dtype, const Shape **s)
{
    *s = dtype == NSK_BF16 ? kBf16 : kF32;
    return 3;
}

// Shape and number of splits by cost: rounds of blocks on the 256 CUs, and the partial sums written and read again.
int choose(int dtype, int L, int K, int NT, int groups, int *splits, int *rows)
{
    const Shape *s;
    const int n = shapes(dtype, &s);
    const int forced = hooks().igemm_tile;   // NSK_IGEMM_TILE = 1.. (test hook)
    int best = 0;
    double best_cost = -1;
    for (int i = 0; i < n; ++i) {
        if (forced >= 1 && (forced - 1) % n != i) continue;
        const long tiles = (long)ceil_div(K, s[i].bm) * ceil_div(NT, s[i].bn) * groups;
        const int nk = ceil_div(L, s[i].kt);
        const bool pieces = s[i].pieces;
        for (int blocks = 256; blocks <= 1280; blocks += 256) {
            if (blocks == 1280 && !pieces) continue;
            long sp = blocks == 1280 ? ceil_div(nk, kPieces) : blocks / tiles;      // (pieces: as few splits as they may have, too)
            if (sp < 1) sp = 1;
            if (sp > nk) sp = nk;
            const int per = ceil_div(nk, (int)sp);
            if (pieces && per > kPieces) continue;
            sp = ceil_div(nk, per);
            const double rounds = (double)((tiles * sp + 255) / 256);
            // 1900 clk/us; 4 TB/s for the partial sums in both directions
            const double cost = s[i].fixed + rounds * (per * (rounds > 1 ? s[i].step : s[i].alone) + s[i].rest) + (sp > 1 ? (double)sp * K * groups * NT * 8 / 4e6 * 1900 + 6000 : 0);
            if (best_cost < 0 || cost < best_cost) {
                best = i;
                best_cost = cost;
                *splits = (int)sp;
                *rows = per * s[i].kt;
            }
        }
    }
    return best;
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int KT, int ST, int CH> int launch(const WgradArgs &a, hipStream_t stream)
{
    PipeArgs w{};
    w.g = a;
    w.by_pq = make_div(a.P * a.Q);
    w.by_q = make_div(a.Q);
    w.tiles_n = ceil_div(a.ntaps * a.C, BN);
    w.tiles_k = ceil_div(a.K, BM);
    w.x_bytes = (unsigned)((long long)a.Nimg * a.H * a.W * a.ldx * (int)sizeof(T));
    w.dy_bytes = (unsigned)((long long)a.L * a.ldy * (int)sizeof(T));
    hipLaunchKernelGGL((wgrad_pipe_kernel<T, BM, BN, WM, WN, WK, KT, ST, CH>), dim3((unsigned)(w.tiles_n * w.tiles_k * a.splits), 1, a.groups),
                       dim3(64 * WM * WN * WK), 0, stream, w);
    return check_launch();
}

}  // namespace

// C and K of one group, ld = channels between two pixels.  (P*Q and the tensors' bytes are within 32 bits for every
// descriptor the library takes.)
bool wgrad_pipe_applicable(int dtype, int C, int K, int groups)
{
    const int vec = dtype == NSK_BF16 ? 8 : 4;
    return C % vec == 0 && K % vec == 0 && groups <= 65535;
}

int wgrad_pipe_rows_per_split(int dtype, int L, int K, int ntapsC, int groups, int *splits)
{
    int rows;
    choose(dtype, L, K, ntapsC, groups, splits, &rows);
    return rows;
}

// groups, ldx, ldy set
int launch_wgrad_pipe(int dtype, const WgradArgs &a, hipStream_t stream)
{
    int splits, rows;
    const int i = choose(dtype, a.L, a.K, a.ntaps * a.C, a.groups, &splits, &rows);
    if (splits != a.splits || rows != a.rows_per_split) return NSK_ERR_BAD_DESC;
    if (dtype != NSK_BF16) {
        switch (i) {
        case 0: return launch<float, 64, 64, 2, 2, 1, 32, 4, 2>(a, stream);
        case 1: return launch<float, 64, 128, 1, 2, 2, 32, 3, 1>(a, stream);
        default: return launch<float, 128, 128, 2, 2, 2, 32, 3, 1>(a, stream);
        }
    }
    const bool is_long = rows > kLong * 64;
    switch (i) {
    case 0: return is_long ? launch<bf16_t, 128, 128, 2, 4, 1, 64, 4, 1>(a, stream) : launch<bf16_t, 128, 128, 2, 4, 1, 64, 4, 2>(a, stream);
    case 1: return is_long ? launch<bf16_t, 64, 128, 2, 4, 1, 64, 4, 1>(a, stream) : launch<bf16_t, 64, 128, 2, 4, 1, 64, 4, 2>(a, stream);
    default: return is_long ? launch<bf16_t, 64, 64, 2, 2, 1, 64, 3, 1>(a, stream) : launch<bf16_t, 64, 64, 2, 2, 1, 64, 3, 2>(a, stream);
    }
}

}  // namespace nsk
