// Implicit-GEMM convolution on the MFMA units of gfx950: the dispatch of conv forward and backward-data to their kernels,
// and the kernel for channel counts that no 16-byte load fits (both passes are "gather a shifted activation tile,
// multiply by a packed filter").
//
// GEMM view (the forward pass of a convolution layer of the ResNet recipe the paper trains,
// section "Experiments and Discussion"): rows m = output pixels, columns n = output channels,
// reduction k = (filter tap, input channel).  In NHWC each tap is a contiguous run of channels, and no im2col buffer
// ever exists in memory.
//
// The element-wise kernel: 256 threads = 4 wavefronts per block, block tile BM x BN, k-tile of 64 bytes per row, staged
// through LDS (rows padded to 80 bytes so the 16-byte fragment reads of 8 consecutive lanes cover all 32 banks once) with
// register prefetch of the next k-tile and two LDS buffers, so one barrier per k-tile suffices.  Each wavefront owns a
// WM x WN sub-tile made of 32x32 MFMA accumulators.
#include <stdlib.h>

#include "nsk_internal.h"

namespace nsk {
namespace {

// BKB = bytes of reduction index per k-tile row (64 or 128); LDS rows are padded by 16 bytes so
// that the 16-byte fragment reads of 8 consecutive rows fall into 8 different bank groups.
template <typename T> struct Traits;
template <> struct Traits<float> {
    static constexpr int VEC = 4;
    typedef f32x4 Vec;
};
template <> struct Traits<bf16_t> {
    static constexpr int VEC = 8;
    typedef bf16x8 Vec;
};

template <typename Vec> __device__ inline Vec zero_vec()
{
    Vec v;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(Vec) / sizeof(v[0])); ++i) v[i] = 0;
    return v;
}

__device__ inline float to_float(float v) { return v; }
__device__ inline float to_float(bf16_t v) { return (float)v; }

template <typename T, int BM, int BN, int WM, int WN, int BKB>
__global__ __launch_bounds__(256) void igemm_kernel(const IgemmArgs a)
{
    typedef Traits<T> TR;
    typedef typename TR::Vec Vec;
    constexpr int VEC = TR::VEC, BK = BKB / (int)sizeof(T), LDK = BK + VEC;
    constexpr int WAVES_N = BN / WN;
    static_assert((BM / WM) * WAVES_N == 4, "four wavefronts per block");
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int VPR = BK / VEC;        // 16-byte vectors per tile row
    constexpr int RPP = 256 / VPR;       // tile rows loaded per pass of the 256 threads
    constexpr int A_PASSES = BM / RPP;
    constexpr int B_PASSES = (BN + RPP - 1) / RPP;

    __shared__ __attribute__((aligned(16))) T smem_ab[2 * (BM + BN) * LDK];
    T(*As)[BM * LDK] = (T(*)[BM * LDK])smem_ab;
    T(*Bs)[BN * LDK] = (T(*)[BN * LDK])(smem_ab + 2 * BM * LDK);
    __shared__ long out_off[BM];
    __shared__ short s_offh[kMaxTaps], s_offw[kMaxTaps];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int m0 = blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    // grouped convolution: blockIdx.z names the group (0 for a plain launch); ld = channels between two source pixels
    const int grp = blockIdx.z, ld = a.src_ld;
    const int src_c0 = grp * a.Cs;            // first source channel of the group
    const long wrow0 = (long)grp * a.Ngemm;   // first filter row = first output channel of the group

    if (tid < kMaxTaps) {
        s_offh[tid] = a.off_h[tid];
        s_offw[tid] = a.off_w[tid];
    }

    const T *__restrict__ src = (const T *)a.src;
    const T *__restrict__ wpk = (const T *)a.wpk;

    // Each thread gathers the same rows in every k-tile: decode them once.
    const int kv = tid % VPR;  // which 16-byte vector of the k-tile row
    const int r0 = tid / VPR;  // row within a pass of RPP rows
    int a_img[A_PASSES], a_bh[A_PASSES], a_bw[A_PASSES];
    bool a_ok[A_PASSES];
#pragma unroll
    for (int u = 0; u < A_PASSES; ++u) {
        const int row = r0 + RPP * u;
        const int m = m0 + row;
        a_ok[u] = m < a.M;
        const int mm = a_ok[u] ? m : 0;
        const int per_img = a.Mi * a.Mj;
        const int img = mm / per_img;
        const int rem = mm - img * per_img;
        const int i = rem / a.Mj;
        const int j = rem - i * a.Mj;
        a_img[u] = img * a.Hs;
        a_bh[u] = i * a.mult_h + a.add_h;
        a_bw[u] = j * a.mult_w + a.add_w;
        if (kv == 0)
            out_off[row] = a_ok[u] ? (((long)img * a.Ho + (i * a.osh + a.oa)) * a.Wo + (j * a.osw + a.ob)) * a.Co + wrow0
                                   : -1L;
    }
    __syncthreads();
    Vec ra[A_PASSES], rb[B_PASSES];

    auto load_tile = [&](int kt) {
        const int kk = kt * BK + kv * VEC;
        // Element-wise gather for channel counts that are not a multiple of the vector width
        // (the 3-channel image stem).
#pragma unroll
        for (int u = 0; u < A_PASSES; ++u) ra[u] = zero_vec<Vec>();
#pragma unroll
        for (int u = 0; u < B_PASSES; ++u) rb[u] = zero_vec<Vec>();
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const int k = kk + e;
            if (k < a.Ktot) {
                const int tap = k / a.Cs;
                const int c = k - tap * a.Cs;
                const int oh = s_offh[tap], ow = s_offw[tap];
#pragma unroll
                for (int u = 0; u < A_PASSES; ++u) {
                    const int h = a_bh[u] + oh, w = a_bw[u] + ow;
                    const bool ok = a_ok[u] && (unsigned)h < (unsigned)a.Hs && (unsigned)w < (unsigned)a.Ws;
                    if (ok) ra[u][e] = src[((long)(a_img[u] + h) * a.Ws + w) * ld + src_c0 + c];
                }
#pragma unroll
                for (int u = 0; u < B_PASSES; ++u) {
                    const int row = r0 + RPP * u;
                    const int n = n0 + row;
                    if (row < BN && n < a.Ngemm) rb[u][e] = wpk[(wrow0 + n) * a.Ktot + k];
                }
            }
        }
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int u = 0; u < A_PASSES; ++u) *(Vec *)&As[buf][(r0 + RPP * u) * LDK + kv * VEC] = ra[u];
#pragma unroll
        for (int u = 0; u < B_PASSES; ++u) {
            const int row = r0 + RPP * u;
            if (row < BN) *(Vec *)&Bs[buf][row * LDK + kv * VEC] = rb[u];
        }
    };

    // The filter rows are the MFMA "A" operand and the pixels the "B" operand, so a lane ends up with 4
    // CONSECUTIVE CHANNELS of one pixel per accumulator quad: acc[mi][ni][4g+j] is channel
    // 32*ni + 8*g + 4*(lane/32) + j of pixel 32*mi + lane%32 of the wavefront's sub-tile.
    const int frow = lane & 31, fk = lane >> 5;
    T *__restrict__ out = (T *)a.out;
    const int wcol0 = n0 + wn * WN;   // first output channel of this wavefront
    f32x16 acc[FM][FN];
#pragma unroll
    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
        for (int ni = 0; ni < FN; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    if (a.accumulate && a.vec_out) {
        // start from the old values: the sum is then rounded to the storage type exactly once
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
            const long off = out_off[wm * WM + mi * 32 + frow];
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int col = wcol0 + ni * 32 + g * 8 + fk * 4;
                    if (off >= 0 && col < a.Ngemm) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[mi][ni][g * 4 + j] = to_float(out[off + col + j]);
                    }
                }
        }
    }

    const int nk = (a.Ktot + BK - 1) / BK;
    if (nk > 0) {
        load_tile(0);
        store_tile(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_tile(kt + 1);
        const T *pa = &As[buf][(wm * WM + frow) * LDK + fk * VEC];
        const T *pb = &Bs[buf][(wn * WN + frow) * LDK + fk * VEC];
#pragma unroll
        for (int ks = 0; ks < BK; ks += 2 * VEC) {
            Vec af[FM], bfv[FN];
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) af[mi] = *(const Vec *)(pa + mi * 32 * LDK + ks);
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) bfv[ni] = *(const Vec *)(pb + ni * 32 * LDK + ks);
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < FN; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfv[ni], af[mi], acc[mi][ni], 0, 0, 0);
            } else {
                // Lane (row, half) holds k = 4*half + t of this group of 8; the same map is used
                // for both operands, so the four steps together cover the 8 k exactly once.
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                        for (int ni = 0; ni < FN; ++ni)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(bfv[ni][t], af[mi][t], acc[mi][ni], 0, 0, 0);
            }
        }
        if (kt + 1 < nk) store_tile(buf ^ 1);
        __syncthreads();
    }

    if (a.vec_out) {
        // Round to the storage type, transpose one 32 x 32 accumulator tile at a time through this
        // wavefront's strip of the (now idle) operand buffers, and store 16 contiguous bytes per lane.
        typedef T T4 __attribute__((ext_vector_type(4)));
        constexpr int SROW = 32 * (int)sizeof(T) + 16;      // staged bytes per pixel (padded)
        constexpr int CPP = 32 * (int)sizeof(T) / 16;       // 16-byte chunks per pixel
        static_assert(4 * 32 * SROW <= (int)sizeof(smem_ab), "epilogue staging fits in the operand buffers");
        unsigned char *my_st = (unsigned char *)smem_ab + wave * (32 * SROW);
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    T4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j) pk[j] = (T)acc[mi][ni][g * 4 + j];
                    *(T4 *)(my_st + frow * SROW + (g * 8 + fk * 4) * (int)sizeof(T)) = pk;
                }
#pragma unroll
                for (int jj = 0; jj < 32 * CPP / 64; ++jj) {
                    const int idx = lane + 64 * jj, pos = idx / CPP, ck = idx % CPP;
                    const Vec v = *(const Vec *)(my_st + pos * SROW + ck * 16);
                    const long off = out_off[wm * WM + mi * 32 + pos];
                    const int col = wcol0 + ni * 32 + ck * VEC;
                    if (off >= 0 && col < a.Ngemm) *(Vec *)(out + off + col) = v;
                }
            }
    } else {
        // element-wise stores (output rows that are not 16-byte granular)
#pragma unroll
        for (int mi = 0; mi < FM; ++mi) {
            const long off = out_off[wm * WM + mi * 32 + frow];
            if (off < 0) continue;
#pragma unroll
            for (int ni = 0; ni < FN; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int col = wcol0 + ni * 32 + 8 * (v >> 2) + 4 * fk + (v & 3);
                    if (col < a.Ngemm) {
                        float r = acc[mi][ni][v];
                        if (a.accumulate) r += to_float(out[off + col]);
                        out[off + col] = (T)r;
                    }
                }
        }
    }
}

template <typename T, int BM, int BN, int WM, int WN, int BKB>
int launch_tile(const IgemmArgs &a, hipStream_t stream)
{
    dim3 grid(ceil_div(a.M, BM), ceil_div(a.Ngemm, BN), a.groups);
    hipLaunchKernelGGL((igemm_kernel<T, BM, BN, WM, WN, BKB>), grid, dim3(256), 0, stream, a);
    return check_launch();
}

// What the output rows are made of: whole 16-byte vectors (1), whole 8-byte ones (2, bf16), neither (0).
int output_vectors(int dtype, const IgemmArgs &a)
{
    const int vec = dtype == NSK_BF16 ? 8 : 4;
    if ((uintptr_t)a.out % 16 != 0 || a.Ngemm % 4 != 0 || a.Co % 4 != 0) return 0;
    return a.Ngemm % vec == 0 && a.Co % vec == 0 ? 1 : 2;
}

// Channel runs and filter rows on 16-byte boundaries: the pipelined kernel takes the launch.  (For a grouped launch
// Cs % VEC == 0 also puts every group's channel run and filter rows on such boundaries.)
bool vector_runs(int dtype, const IgemmArgs &a)
{
    const int vec = dtype == NSK_BF16 ? 8 : 4, ld = a.groups > 1 ? a.src_ld : a.Cs;
    return a.Cs % vec == 0 && ld % vec == 0 && a.Ktot % vec == 0 && ((uintptr_t)a.src % 16 == 0) && ((uintptr_t)a.wpk % 16 == 0);
}

// Tile of the element-wise kernel: 0 = 256x32 (64-row wavefront tiles), 1 = 128x64 (32-row), 2 = 128x128 (64-row).
int auto_tile(const IgemmArgs &a, int es)
{
    if (a.Ngemm <= 32) return 0;
    if (a.Ngemm <= 64) return 1;
    if ((long)a.Ktot * es >= 1024) return 2;
    return 1;
}

template <typename T> int launch_typed(const IgemmArgs &a, hipStream_t stream)
{
    // Measured on MI355X: with 64 or fewer columns the 128-row tile wins (more blocks in flight hide
    // the per-block prologue and epilogue); wide problems with a long reduction take 128x128 tiles.
    switch (auto_tile(a, (int)sizeof(T))) {
    case 0: return launch_tile<T, 256, 32, 64, 32, 64>(a, stream);
    case 1: return launch_tile<T, 128, 64, 32, 64, 64>(a, stream);
    default: return launch_tile<T, 128, 128, 64, 64, 64>(a, stream);
    }
}

}  // namespace

int igemm_stats_rows(int dtype, const IgemmArgs &a)
{
    // the same order of tests as launch_igemm
    if (a.M <= 0 || a.Ngemm <= 0 || a.accumulate) return 0;
    if (a.groups > 1) return 0;
    const bool special = hooks().igemm_tile == 0;
    if (special) {
        if (tiny_src_applicable(dtype, a) || tiny_out_applicable(dtype, a)) return 0;   // no statistics epilogue there
        if (halo64_applicable(dtype, a)) return halo64_stats_rows(a);
        if (fs64_fwd_s2_applicable(dtype, a)) return fs64_fwd_s2_stats_rows(a);
        if (conv_pw_applicable(dtype, a)) return conv_pw_stats_rows(a);
        if (halo_wide_applicable(dtype, a)) return halo_wide_stats_rows(a);
        if (halo_wide_fwd_s2_applicable(dtype, a)) return halo_wide_fwd_s2_stats_rows(a);
    }
    // The pipelined kernel needs 16-byte stores of the partial sums; one or two rows for every row block.  Its epilogue beats
    // the separate pass over y at every size (us, convolution + batch-norm, pass / epilogue: 256->1024 1x1 at 14x14 N=128
    // 69.6 / 69.4, 64->128 1x1 stride 2 at 56x56 N=64 29.2 / 25.1, fp32 16->16 at 40x42 N=37 22.5 / 20.8, 72->104 at 29x37
    // N=20 34.0 / 20.5; 256->64 at 56x56 N=64, 3136 rows of sums, 50.1 / 51.5).
    return output_vectors(dtype, a) != 0 && vector_runs(dtype, a) ? igemm_pipe_stats_rows(dtype, a) : 0;
}

// The residue classes of a strided backward-data pass in one launch of the pipelined kernel, if it is what each of them runs on.
bool igemm_pipe_multi_applicable(int dtype, const IgemmArgs *a, int count)
{
    for (int i = 0; i < count; ++i) {
        if (a[i].zero_cell || a[i].stats || !vector_runs(dtype, a[i])) return false;
        if (a[i].groups > 1 && !hooks().no_depthwise && hooks().igemm_tile == 0 && depthwise_applicable(dtype, a[i])) return false;
        if (a[i].groups <= 1 && hooks().igemm_tile == 0 &&
            (tiny_src_applicable(dtype, a[i]) || tiny_out_applicable(dtype, a[i]) || (count == 1 && conv_pw_applicable(dtype, a[i]))))
            return false;   // (several classes in one launch beat the short-reduction kernel's one launch each: 3x3 stride 2 32->64 17.4 / 8.6 us)
    }
    return count >= 1 && count <= 4;
}

int launch_igemm_pipe_multi(int dtype, const IgemmArgs *a, int count, hipStream_t stream)
{
    IgemmArgs b[4];
    for (int i = 0; i < count; ++i) {
        b[i] = a[i];
        if (b[i].groups <= 1) {
            b[i].groups = 1;
            b[i].src_ld = b[i].Cs;
        }
        b[i].vec_out = output_vectors(dtype, b[i]);
    }
    return launch_igemm_pipe(dtype, b, count, stream);
}

int launch_igemm(int dtype, const IgemmArgs &a, hipStream_t stream)
{
    if (a.M <= 0 || a.Ngemm <= 0) return NSK_OK;
    const bool grouped = a.groups > 1;   // only the generic kernel knows about groups
    if (grouped && (a.groups > 65535 || a.src_ld != a.groups * a.Cs || a.zero_cell || a.stats)) return NSK_ERR_BAD_DESC;
    if (a.zero_cell) return launch_conv_pw(a, stream);   // the caller has checked that this kernel applies
    const bool special = hooks().igemm_tile == 0 && !grouped;   // (the variable is a test hook)
    if (special && tiny_src_applicable(dtype, a)) return launch_tiny_src(dtype, a, stream);
    if (special && tiny_out_applicable(dtype, a)) return launch_tiny_out(dtype, a, stream);
    if (special && halo64_applicable(dtype, a)) return launch_halo64(a, stream);
    if (special && fs64_fwd_s2_applicable(dtype, a)) return launch_fs64_fwd_s2(a, stream);
    if (special && conv_pw_applicable(dtype, a)) return launch_conv_pw(a, stream);
    if (special && halo_wide_applicable(dtype, a)) return launch_halo_wide(a, stream);
    if (special && halo_wide_fwd_s2_applicable(dtype, a)) return launch_halo_wide_fwd_s2(a, stream);
    if (grouped && hooks().igemm_tile == 0 && grouped8_applicable(dtype, a)) return launch_grouped8(a, stream);
    if (grouped && hooks().igemm_tile == 0 && !hooks().no_depthwise && depthwise_applicable(dtype, a))
        return launch_depthwise(dtype, a, stream);
    IgemmArgs b = a;
    if (!grouped) {
        b.groups = 1;
        b.src_ld = b.Cs;
    }
    b.vec_out = output_vectors(dtype, b);
    if (vector_runs(dtype, b)) return launch_igemm_pipe(dtype, &b, 1, stream);
    if (b.stats) return NSK_ERR_BAD_DESC;   // (igemm_stats_rows named none)
    b.vec_out = b.vec_out == 1 ? 1 : 0;
    return dtype == NSK_BF16 ? launch_typed<bf16_t>(b, stream) : launch_typed<float>(b, stream);
}

}  // namespace nsk
