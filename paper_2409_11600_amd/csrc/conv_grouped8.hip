// Grouped 3x3 stride-1 layers with eight channels per group on both sides, bf16 (32 groups of 8 and their like): forward,
// backward-data and backward-weight on the matrix units; and backward-weight of plain layers with 16 channels, by the same means.
//
// What bounds them: memory (the contraction is 72 indices long).  The direct kernels of conv_depthwise.hip do 2 x 72
// two-element dot products per eight outputs and read every input vector nine times through the L1: 84 us per data pass
// and 153 us backward-weight for 256 channels at 28x28, N=128, whose operands stream in 20 us.  Here a strip of image
// rows with its halo is copied into LDS once (straight from memory, 16 bytes per lane) and a 16x16x32 MFMA takes one
// filter row of one group: its 32 reduction indices are four pixels x eight channels, exactly the 16-byte pieces a
// lane reads, so nothing is shuffled.  Half of the matrix unit idles (eight output channels, three of four pixels),
// which at 5 us of MFMA time does not matter.  No zero weight ever meets a real pixel (the fourth pixel is read from a
// row of zeros, and so is everything past the end of a strip), so infinities stay where they belong.
//
// Measured (us, 256 channels at 28x28, N=128; direct kernels -> these): forward and backward-data 84.6 -> 25 (107 MB:
// 4.3 TB/s; 14x14x512 16.2 -> 13.1 with eight wavefronts a block for four), backward-weight 153.5 + 8.2 -> 29.5 + 4.7.
//
// Work: a block is 64 channels (eight groups, two per wavefront) of a strip of full image rows.
#include "nsk_internal.h"

namespace nsk {
namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Eight wavefronts: four take two groups each, on every other run of pixels.  A run is a chain (addresses, LDS, three products,
// rounding) that four wavefronts a block, two blocks a CU, do not fill (two runs at a time in four wavefronts 32.8 us, one 33.7,
// eight wavefronts 31.4; sixteen 30.8, but 15.2 against 13.2 at 14x14).
constexpr int G8_THREADS = 512;
constexpr int G8_ENTRIES = 480;        // pixels of a strip with halo: 60 KB of LDS, two blocks per CU
constexpr int G8_WG_ENTRIES = 600;     // backward-weight: with the strip of dy 75 KB, two blocks per CU

struct G8Args {
    const void *src, *wpk;
    void *out;
    int H, W, C, rows, strips, chunks;     // rows of a strip, strips of an image, 64-channel chunks
    unsigned src_bytes, wpk_bytes, out_bytes;
    unsigned long long taps;               // tap of window position 3*r + s, four bits each
    Div by_pw, by_w;                       // W + 2, W
};

// The strip with its halo, rows of eight 16-byte pieces per pixel: piece p of entry e lies at p ^ swap(e).
template <int WAVES, typename F> __device__ inline void stage(__amdgpu_buffer_rsrc_t rsrc, unsigned char *lds, int entries, int wave, int lane, F offset_of)
{
    for (int i = wave; i * 8 < entries; i += WAVES) {
        const int e = i * 8 + (lane >> 3);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(lds + i * 1024), 16, (int)offset_of(e, lane & 7), 0, 0, 0);
    }
}

// every wavefront's direct loads and LDS writes have arrived
__device__ inline void direct_loads_done()
{
    __builtin_amdgcn_s_waitcnt(7 << 4);
    __syncthreads();
}

template <bool ACC> __global__ __launch_bounds__(G8_THREADS) void grouped8_kernel(const G8Args a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int mover = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wave = mover & 3;
    const int chunk = blockIdx.x % a.chunks, rest = blockIdx.x / a.chunks;
    const int strip = rest % a.strips, img = rest / a.strips;
    const int h0 = strip * a.rows, rows = min(a.rows, a.H - h0), PW = a.W + 2;
    const int entries = (rows + 2) * PW, zero = (entries + 7) & ~7;
    const __amdgpu_buffer_rsrc_t src_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.src, 0, a.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wpk_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.wpk, 0, a.wpk_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t out_rsrc = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, a.out_bytes, 0x00020000);
    // sixteen neighbouring pixels are read at once: their pieces are exchanged so that they cover all banks
    stage<G8_THREADS / 64>(src_rsrc, smem, entries, mover, lane, [&](int e, int slot) {
        const int er = divide(e, a.by_pw), h = h0 - 1 + er, w = e - er * PW - 1;
        const int ch = chunk * 64 + ((slot ^ (e >> 1)) & 7) * 8;
        const unsigned bad = (unsigned)((h | (a.H - 1 - h) | w | (a.W - 1 - w) | (a.C - 1 - ch) | (entries - 1 - e)) >> 31);
        return ((unsigned)(((img * a.H + h) * a.W + w) * a.C + ch) * 2u) | bad;
    });
    if (threadIdx.x < 8) *(f32x4 *)(smem + zero * 128 + threadIdx.x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};

    // filter rows: lane (output channel m = lane % 16, window column c = lane / 16) holds the eight input channels
    const int m = lane & 15, c = lane >> 4;
    bf16x8 wf[2][3];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int k = chunk * 64 + (wave * 2 + g) * 8 + m;
            const unsigned tap = (unsigned)(a.taps >> (4 * (3 * r + (c < 3 ? c : 0)))) & 15u;
            const unsigned at = (m < 8 && c < 3 && k < a.C) ? (unsigned)(k * 72 + tap * 8) * 2u : ~0u;
            wf[g][r] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wpk_rsrc, (int)at, 0, 0));
        }
    direct_loads_done();

    const int pixels = rows * a.W;
    const int ch = chunk * 64 + wave * 16 + (c & 1) * 4;                     // of the first group's results
    const unsigned pix0 = (unsigned)((img * a.H + h0) * a.W);
    const int first = chunk * 64 + wave * 16 + (c & 1) * 8;                  // of the channels that this lane stores
    for (int l0 = (mover >> 2) * 16; l0 < pixels; l0 += G8_THREADS / 256 * 16) {
        const int l = l0 + m, row = divide(l, a.by_w), e0 = row * PW + (l - row * a.W) + c;
        const bool real = c < 3 && l < pixels;
        const unsigned pixel = (pix0 + (unsigned)l) * (unsigned)a.C;
        f32x4 acc[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (ACC) {     // start from the old values: one rounding
                const unsigned at = c < 2 && l < pixels && ch + 8 * g < a.C ? (pixel + (unsigned)(ch + 8 * g)) * 2u : ~0u;
                const bf16x4 old = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(out_rsrc, (int)at, 0, 0));
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[g][j] = (float)old[j];
            }
        }
        bf16x8 b[3][2];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int e = real ? e0 + r * PW : zero;
            const unsigned char *p = smem + e * 128 + (((wave * 2) ^ (e >> 1)) & 7) * 16;
            b[r][0] = *(const bf16x8 *)p;
            b[r][1] = *(const bf16x8 *)(smem + ((unsigned)(p - smem) ^ 16u));
        }
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int g = 0; g < 2; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[g][r], b[r][g], acc[g], 0, 0, 0);
        // lane (pixel, quarter): rows 4*quarter .. of the result; quarters 2 and 3 hold nothing.  The halves of the two groups change
        // places between quarters 0 and 1, so that a lane stores the eight channels of one group: a pixel's 32 bytes from this
        // wavefront in one instruction
        u32x2 o[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            bf16x4 r;
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = (bf16_t)acc[g][j];
            o[g] = __builtin_bit_cast(u32x2, r);
        }
        const u32x2 lo = __builtin_amdgcn_permlane16_swap(o[0][0], o[1][0], false, false);
        const u32x2 hi = __builtin_amdgcn_permlane16_swap(o[0][1], o[1][1], false, false);
        const unsigned to = c < 2 && l < pixels && first < a.C ? (pixel + (unsigned)first) * 2u : ~0u;
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{lo[0], hi[0], lo[1], hi[1]}, out_rsrc, (int)to, 0, 0);
    }
}

// ---- backward-weight: dw[k][tap][c] of a group = sum over pixels of dy[pixel][k] * x[pixel + tap][c].  A wavefront takes two
// groups: rows of the MFMA = their sixteen dy channels, columns = their sixteen x channels of one tap (the two off-diagonal
// blocks are not stored), reduction = 32 consecutive pixels of the strip, through the transposing LDS read.
// The vector unit's addresses bounded it (0.87 of the clocks), so a pixel's pieces are swapped by two neighbouring bits of its index, which an AND
// of its shifted byte offset yields, and runs whose 32 pixels are all there have no choice between a place and the zeros: 190 -> 113 instructions a
// run, 37.9 -> 29.5 us for 128 images of 28x28x256, 123 MB.
struct G8WArgs {
    const void *x, *dy;
    float *part;
    int H, W, C, rows, strips, chunks, tiles, splits;
    unsigned x_bytes, dy_bytes;
    unsigned long long taps;
    Div by_pw, by_w, by_strips;
};

// within 32 lanes a transposing read serves eight consecutive pixels, 32 bytes each: spread over all banks
__device__ inline int g8_swap(int e) { return e & 6; }

__global__ __launch_bounds__(G8_THREADS) void grouped8_wgrad_kernel(const G8WArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int mover = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wave = mover & 3, half = mover >> 2;
    const int chunk = blockIdx.x % a.chunks, split = blockIdx.x / a.chunks, PW = a.W + 2;
    const int dy_at = (((a.rows + 2) * PW + 7) & ~7) * 128, zero = dy_at + ((a.rows * a.W + 7) & ~7) * 128;   // bytes
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t dy_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.dy, 0, a.dy_bytes, 0x00020000);
    if (threadIdx.x < 8) *(f32x4 *)(smem + zero + threadIdx.x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};

    const int q = lane >> 4, i16 = lane & 15;
    const int inner = (i16 & 1) * 8, mine = (wave * 2 + ((i16 & 3) >> 1)) * 16 + inner;   // a lane's place in a pixel before the swap
    f32x4 sum[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tile = split; tile < a.tiles; tile += a.splits) {
        const int img = divide(tile, a.by_strips), h0 = (tile - img * a.strips) * a.rows, rows = min(a.rows, a.H - h0);
        const int entries = (rows + 2) * PW, pixels = rows * a.W;
        __syncthreads();   // everybody has read the strip before
        for (int i = mover; i * 8 < entries; i += G8_THREADS / 64) {
            const int e = i * 8 + (lane >> 3), er = divide(e, a.by_pw), h = h0 - 1 + er, w = e - er * PW - 1;
            const int ch = chunk * 64 + ((lane & 7) ^ g8_swap(e)) * 8;
            const unsigned bad = (unsigned)((h | (a.H - 1 - h) | w | (a.W - 1 - w) | (a.C - 1 - ch) | (entries - 1 - e)) >> 31);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void *)(smem + i * 1024), 16,
                                                     (int)(((unsigned)(((img * a.H + h) * a.W + w) * a.C + ch) * 2u) | bad), 0, 0, 0);
        }
        for (int i = mover; i * 8 < pixels; i += G8_THREADS / 64) {
            const int e = i * 8 + (lane >> 3);
            const int ch = chunk * 64 + ((lane & 7) ^ g8_swap(e)) * 8;
            const unsigned bad = (unsigned)(((a.C - 1 - ch) | (pixels - 1 - e)) >> 31);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(dy_rsrc, (lds_void *)(smem + dy_at + i * 1024), 16,
                                                     (int)(((unsigned)(((img * a.H + h0) * a.W + e) * a.C + ch) * 2u) | bad), 0, 0, 0);
        }
        direct_loads_done();
        f32x4 acc[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        // 32 pixels; FULL: all of them are there, and no read has to choose between its place and the zeros
        auto run = [&](auto full, int l0) {
            constexpr bool FULL = decltype(full)::value;
            bf16x4 d[2];
            int e[2];                                      // bytes
            bool real[2];
            auto read = [&](int pixel, int base, bool is_real) {
                const int at = ((pixel >> 3 & 96) ^ mine) + pixel + base;
                return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(smem + (FULL || is_real ? at : zero + inner)));
            };
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int l = l0 + 16 * hi + 4 * q + (i16 >> 2), row = divide(l, a.by_w);
                real[hi] = l < pixels;
                e[hi] = (l + row * 2) * 128;               // (a row of x has two pixels more)
                d[hi] = read(l * 128, dy_at, real[hi]);
            }
            const bf16x8 af = __builtin_shufflevector(d[0], d[1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                bf16x4 b[2];
#pragma unroll
                for (int hi = 0; hi < 2; ++hi) b[hi] = read(e[hi] + ((t / 3) * PW + t % 3) * 128, 0, real[hi]);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, __builtin_shufflevector(b[0], b[1], 0, 1, 2, 3, 4, 5, 6, 7), acc[t], 0, 0, 0);
            }
        };
        int l0 = 32 * half;
        for (; l0 + 32 <= pixels; l0 += 64) run(std::true_type{}, l0);
        if (l0 < pixels) run(std::false_type{}, l0);
#pragma unroll
        for (int t = 0; t < 9; ++t) sum[t] += acc[t];      // (a strip's sum at a time: the chains stay short)
    }
    // the second four wavefronts' sums through LDS
    __syncthreads();
    f32x4 *const other = (f32x4 *)smem + (size_t)(wave * 64 + lane);
    if (half) {
#pragma unroll
        for (int t = 0; t < 9; ++t) other[t * 256] = sum[t];
    }
    __syncthreads();
    if (half) return;
#pragma unroll
    for (int t = 0; t < 9; ++t) sum[t] += other[t * 256];
    // result rows 4*q + j = dy channel, column i16 = x channel of the wavefront's sixteen: same group on the diagonal blocks
    if ((q >> 1) == (i16 >> 3)) {
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int tap = (int)(a.taps >> (4 * t)) & 15;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = chunk * 64 + wave * 16 + 4 * q + j;
                if (k < a.C) a.part[((size_t)split * a.C + k) * 72 + tap * 8 + (i16 & 7)] = sum[t][j];
            }
        }
    }
}

// ---- backward-weight of plain layers with 16 channels in and out: a wavefront's product above is then the layer's own, and the
// pipelined split-K kernel, which stages every pixel of x once per tap and fills a quarter of its 64 rows, is bound by what
// it stages.  Here a strip of x with its halo and the strip of dy lie in LDS once ([pixel][channel], 32 bytes a pixel, so that the
// eight consecutive pixels that a transposing read serves at once are 256 bytes), and the eight wavefronts share the strip's runs
// of 32 pixels.  What is left is a chain: launch, one load of a strip, 40 reads and 18 products a run, the sums through
// LDS.  256 images of 32x32 with the reduction 19.5 -> 12.7 us, 512 images 29.9 -> 15.6 us.  (With 32 channels the partial sums are
// four times as many: 256 images of 16x16 13.7 / 20.4 us, so these layers stay there.)
struct NarrowWArgs {
    const void *x, *dy;
    float *part;
    int H, W, rows, strips, tiles, splits;
    unsigned bytes;
    unsigned long long taps;
    Div by_pw, by_w, by_strips;
};

constexpr int strip16(int entries) { return (entries * 32 + 1023) & ~1023; }     // bytes in LDS: whole direct loads

__global__ __launch_bounds__(G8_THREADS) void narrow_wgrad_kernel(const NarrowWArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), PW = a.W + 2;
    const int dy_at = strip16((a.rows + 2) * PW), zero = dy_at + strip16(a.rows * a.W);   // bytes
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t dy_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.dy, 0, a.bytes, 0x00020000);
    if (threadIdx.x < 2) *(f32x4 *)(smem + zero + threadIdx.x * 16) = f32x4{0.f, 0.f, 0.f, 0.f};

    const int q = lane >> 4, i16 = lane & 15, inner = (i16 & 3) * 8;
    f32x4 sum[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tile = blockIdx.x; tile < a.tiles; tile += a.splits) {
        const int img = divide(tile, a.by_strips), h0 = (tile - img * a.strips) * a.rows, rows = min(a.rows, a.H - h0);
        const int entries = (rows + 2) * PW, pixels = rows * a.W;
        __syncthreads();   // everybody has read the strip before
        for (int i = wave; i * 32 < entries; i += G8_THREADS / 64) {
            const int e = i * 32 + (lane >> 1), er = divide(e, a.by_pw), h = h0 - 1 + er, w = e - er * PW - 1;
            const unsigned bad = (unsigned)((h | (a.H - 1 - h) | w | (a.W - 1 - w) | (entries - 1 - e)) >> 31);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void *)(smem + i * 1024), 16,
                                                     (int)(((unsigned)((img * a.H + h) * a.W + w) * 32u + (lane & 1) * 16u) | bad), 0, 0, 0);
        }
        for (int i = wave; i * 32 < pixels; i += G8_THREADS / 64) {
            const int e = i * 32 + (lane >> 1);
            const unsigned bad = (unsigned)((pixels - 1 - e) >> 31);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(dy_rsrc, (lds_void *)(smem + dy_at + i * 1024), 16,
                                                     (int)(((unsigned)((img * a.H + h0) * a.W + e) * 32u + (lane & 1) * 16u) | bad), 0, 0, 0);
        }
        direct_loads_done();
        f32x4 acc[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int l0 = 32 * wave; l0 < pixels; l0 += G8_THREADS / 2) {
            bf16x4 d[2];
            int e[2];
            bool real[2];
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int l = l0 + 16 * hi + 4 * q + (i16 >> 2), row = divide(l, a.by_w);
                real[hi] = l < pixels;
                e[hi] = row * PW + (l - row * a.W);
                d[hi] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(smem + (real[hi] ? dy_at + l * 32 : zero) + inner));
            }
            const bf16x8 af = __builtin_shufflevector(d[0], d[1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                bf16x4 b[2];
#pragma unroll
                for (int hi = 0; hi < 2; ++hi) {
                    const int at = real[hi] ? (e[hi] + (t / 3) * PW + t % 3) * 32 : zero;
                    b[hi] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(smem + at + inner));
                }
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, __builtin_shufflevector(b[0], b[1], 0, 1, 2, 3, 4, 5, 6, 7), acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 9; ++t) sum[t] += acc[t];      // (a strip's sum at a time: the chains stay short)
    }
    // the wavefronts' sums through LDS: the second four add to the first four, then all threads add up those
    f32x4 *const red = (f32x4 *)smem, *const mine = red + (wave & 3) * 576 + lane;
    __syncthreads();
    if (wave >= 4) {
#pragma unroll
        for (int t = 0; t < 9; ++t) mine[t * 64] = sum[t];
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll
        for (int t = 0; t < 9; ++t) mine[t * 64] += sum[t];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 576; i += G8_THREADS) {
        const f32x4 v = (red[i] + red[576 + i]) + (red[2 * 576 + i] + red[3 * 576 + i]);
        // rows 4 * (lane / 16) + j = dy channel, column lane % 16 = x channel
        const int l = i & 63, tap = (int)(a.taps >> (4 * (i >> 6))) & 15;
        float *const to = a.part + ((size_t)blockIdx.x * 16 + (l >> 4) * 4) * 144 + tap * 16 + (l & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) to[j * 144] = v[j];
    }
}

// Rows of a strip so that `per_row` * rows + `fixed` entries stay within `most`; balanced over the image.
int strip_rows(int H, int per_row, int fixed, int most)
{
    int rows = (most - fixed) / per_row;
    if (rows < 1) return 0;
    if (rows > H) rows = H;
    return ceil_div(H, ceil_div(H, rows));
}

// window position 3*r + s -> tap, four bits each; false if the taps are not the nine of a 3x3 window around the pixel
template <typename A> bool window_taps(const A &a, int add_h, int add_w, unsigned long long *taps)
{
    if (a.ntaps != 9) return false;
    unsigned seen = 0;
    unsigned long long v = 0;
    for (int t = 0; t < 9; ++t) {
        const int eh = add_h + a.off_h[t], ew = add_w + a.off_w[t];
        if (eh < -1 || eh > 1 || ew < -1 || ew > 1) return false;
        const int at = 3 * (eh + 1) + ew + 1;
        seen |= 1u << at;
        v |= (unsigned long long)t << (4 * at);
    }
    *taps = v;
    return seen == 511u;
}

bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool grouped8_applicable(int dtype, const IgemmArgs &a)
{
    unsigned long long taps;
    if (dtype != NSK_BF16 || hooks().no_depthwise || hooks().no_grouped8 || a.groups <= 1 || a.Cs != 8 || a.Ngemm != 8) return false;
    const int C = 8 * a.groups;
    if (a.src_ld != C || a.Co != C || a.Ktot != 72 || a.stats) return false;
    if (a.mult_h != 1 || a.mult_w != 1 || a.osh != 1 || a.osw != 1 || a.oa != 0 || a.ob != 0) return false;
    if (a.Hs != a.Ho || a.Ws != a.Wo || a.Mi != a.Ho || a.Mj != a.Wo) return false;
    return window_taps(a, a.add_h, a.add_w, &taps) && strip_rows(a.Hs, a.Ws + 2, 2 * (a.Ws + 2), G8_ENTRIES) > 0 && al16(a.src) &&
           al16(a.wpk) && al16(a.out);
}

int launch_grouped8(const IgemmArgs &a, hipStream_t stream)
{
    G8Args g{};
    g.src = a.src; g.wpk = a.wpk; g.out = a.out;
    g.H = a.Hs; g.W = a.Ws; g.C = 8 * a.groups;
    g.rows = strip_rows(a.Hs, a.Ws + 2, 2 * (a.Ws + 2), G8_ENTRIES);
    g.strips = ceil_div(a.Hs, g.rows);
    g.chunks = ceil_div(g.C, 64);
    g.src_bytes = a.src_bytes;
    g.wpk_bytes = (unsigned)(g.C * 72 * 2);
    g.out_bytes = (unsigned)((long)a.Nimg * a.Ho * a.Wo * a.Co * 2);
    window_taps(a, a.add_h, a.add_w, &g.taps);
    g.by_pw = make_div(g.W + 2);
    g.by_w = make_div(g.W);
    const size_t smem = (size_t)((((g.rows + 2) * (g.W + 2) + 7) & ~7) + 1) * 128;
    const dim3 grid((unsigned)(a.Nimg * g.strips * g.chunks));
    if (a.accumulate)
        hipLaunchKernelGGL(grouped8_kernel<true>, grid, dim3(G8_THREADS), smem, stream, g);
    else
        hipLaunchKernelGGL(grouped8_kernel<false>, grid, dim3(G8_THREADS), smem, stream, g);
    return check_launch();
}

// groups, ldx, ldy, C = K = 8 of one group
bool grouped8_wgrad_applicable(int dtype, const WgradArgs &a)
{
    unsigned long long taps;
    if (dtype != NSK_BF16 || hooks().no_depthwise || hooks().no_grouped8 || a.groups <= 1 || a.C != 8 || a.K != 8) return false;
    if (a.ldx != 8 * a.groups || a.ldy != 8 * a.groups || a.sh != 1 || a.sw != 1 || a.P != a.H || a.Q != a.W) return false;
    return window_taps(a, -a.ph, -a.pw, &taps) && strip_rows(a.H, 2 * a.W + 2, 2 * (a.W + 2) + 16, G8_WG_ENTRIES) > 0 && al16(a.x) && al16(a.dy);
}

int grouped8_wgrad_splits(const WgradArgs &a)
{
    const int rows = strip_rows(a.H, 2 * a.W + 2, 2 * (a.W + 2) + 16, G8_WG_ENTRIES);
    const int tiles = a.Nimg * ceil_div(a.H, rows);
    // two blocks per CU
    int splits = 512 / ceil_div(8 * a.groups, 64);
    if (splits < 1) splits = 1;
    return splits < tiles ? splits : tiles;
}

int launch_grouped8_wgrad(const WgradArgs &a, hipStream_t stream)
{
    G8WArgs g{};
    g.x = a.x; g.dy = a.dy; g.part = a.part;
    g.H = a.H; g.W = a.W; g.C = 8 * a.groups;
    g.rows = strip_rows(a.H, 2 * a.W + 2, 2 * (a.W + 2) + 16, G8_WG_ENTRIES);
    g.strips = ceil_div(a.H, g.rows);
    g.chunks = ceil_div(g.C, 64);
    g.tiles = a.Nimg * g.strips;
    g.splits = a.splits;
    g.x_bytes = g.dy_bytes = (unsigned)((long)a.Nimg * a.H * a.W * g.C * 2);
    window_taps(a, -a.ph, -a.pw, &g.taps);
    g.by_pw = make_div(g.W + 2);
    g.by_w = make_div(g.W);
    g.by_strips = make_div(g.strips);
    size_t smem = (size_t)((((g.rows + 2) * (g.W + 2) + 7) & ~7) + ((g.rows * g.W + 7) & ~7) + 1) * 128;
    if (smem < 9 * 256 * sizeof(f32x4)) smem = 9 * 256 * sizeof(f32x4);      // the sums of half of the wavefronts
    static std::atomic<unsigned long long> done{0};
    const int rc = allow_lds((const void *)grouped8_wgrad_kernel, 80 * 1024, done);
    if (rc != NSK_OK) return rc;
    hipLaunchKernelGGL(grouped8_wgrad_kernel, dim3((unsigned)(g.chunks * g.splits)), dim3(G8_THREADS), smem, stream, g);
    return check_launch();
}

// Rows of a strip of a plain layer: two blocks' strips fit a CU, and there are no fewer strips than CUs
static int narrow_rows(const WgradArgs &a)
{
    const int rows = strip_rows(a.H, (2 * a.W + 2) * 32, 2 * (a.W + 2) * 32 + 3 * 1024, 78 * 1024), strips = ceil_div(256, a.Nimg);
    return ceil_div(a.H, strips) < rows ? ceil_div(a.H, strips) : rows;
}

// From 65536 pixels in strips of at least 256 on (us with the reduction, here / pipelined kernel: 64 images of 32x32 8.3 / 10.1, 32
// images 8.0 / 7.9, 4 of 112x112 8.5 / 8.7, 256 of 16x16 8.4 / 10.1, 2048 of 8x8 14.4 / 13.1).
bool narrow_wgrad_applicable(int dtype, const WgradArgs &a)
{
    unsigned long long taps;
    if (dtype != NSK_BF16 || a.groups > 1 || a.C != 16 || a.K != 16 || hooks().no_grouped8) return false;
    if (a.sh != 1 || a.sw != 1 || a.P != a.H || a.Q != a.W || (long)a.L * 32 >= 0xF0000000L) return false;
    return window_taps(a, -a.ph, -a.pw, &taps) && a.L >= 65536 && narrow_rows(a) * a.W >= 256 && al16(a.x) && al16(a.dy);
}

// A block a CU; up to 131072 pixels half as many, whose partial sums are half as long (64 images of 32x32 9.0 / 8.3 us, 128 images
// 9.8 / 9.4, 256 images 12.7 / 13.2).
int narrow_wgrad_splits(const WgradArgs &a)
{
    const int tiles = a.Nimg * ceil_div(a.H, narrow_rows(a)), most = a.L <= 131072 ? 128 : 256;
    return tiles < most ? tiles : most;
}

int launch_narrow_wgrad(const WgradArgs &a, hipStream_t stream)
{
    NarrowWArgs g{};
    g.x = a.x; g.dy = a.dy; g.part = a.part;
    g.H = a.H; g.W = a.W;
    g.rows = narrow_rows(a);
    g.strips = ceil_div(a.H, g.rows);
    g.tiles = a.Nimg * g.strips;
    g.splits = a.splits;
    g.bytes = (unsigned)((long)a.L * 32);
    window_taps(a, -a.ph, -a.pw, &g.taps);
    g.by_pw = make_div(g.W + 2);
    g.by_w = make_div(g.W);
    g.by_strips = make_div(g.strips);
    size_t smem = (size_t)strip16((g.rows + 2) * (g.W + 2)) + strip16(g.rows * g.W) + 32;
    if (smem < 4 * 576 * sizeof(f32x4)) smem = 4 * 576 * sizeof(f32x4);      // the sums of half of the wavefronts
    static std::atomic<unsigned long long> done{0};
    const int rc = allow_lds((const void *)narrow_wgrad_kernel, 80 * 1024, done);
    if (rc != NSK_OK) return rc;
    hipLaunchKernelGGL(narrow_wgrad_kernel, dim3((unsigned)g.splits), dim3(G8_THREADS), smem, stream, g);
    return check_launch();
}

}  // namespace nsk
