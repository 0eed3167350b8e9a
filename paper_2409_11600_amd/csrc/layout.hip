// Layout helpers at the library boundary: the kernels compute in NHWC / "filter row = all taps of
// one output channel"; callers that hold NCHW / KCRS tensors are served by these copies through
// the workspace.  Pure data movement, bounded by HBM bandwidth.
#include "nsk_internal.h"

namespace nsk {
namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Per image: src [rows][cols] -> dst [cols][ldo], ldo >= rows (the rest of a row is zeros), 32x32 tiles through LDS (padded
// by one column so the transposed reads are conflict-free).  accumulate adds into dst.
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *__restrict__ src, T *__restrict__ dst, int rows,
                                                        int cols, int ldo, int accumulate)
{
    __shared__ float tile[32][33];
    const long img = blockIdx.z;
    src += img * rows * cols;
    dst += img * ldo * cols;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int r = r0 + ty + i, c = c0 + tx;
        tile[ty + i][tx] = r < rows && c < cols ? (float)src[(long)r * cols + c] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; i += 8) {
        const int c = c0 + ty + i, r = r0 + tx;
        if (r < ldo && c < cols) {
            float v = tile[tx][ty + i];
            T *o = dst + (long)c * ldo + r;
            if (accumulate) v += (float)*o;
            *o = (T)v;
        }
    }
}

struct PackArgs {
    const void *w;
    void *out;
    int Nn, ntaps, Cs, Cr;   // Cr: channels of the source; those from there to Cs are zeros
    long sn, sc;
    long w_gstep;   // grouped filters: blockIdx.z names the group, whose source lies w_gstep elements further
    int tap_off[kMaxTaps];
};

// Up to four packings in one launch (blockIdx.y names the packing): the residue classes of a strided backward-data
// pass each need their own packed filter, and a launch per class costs more than the copy.
constexpr int kPackMulti = 4;
struct PackMulti {
    PackArgs e[kPackMulti];
};

template <typename T> __global__ __launch_bounds__(256) void pack_filter_kernel(const PackMulti m)
{
    const PackArgs &a = m.e[blockIdx.y];
    const long total = (long)a.Nn * a.ntaps * a.Cs;
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int c = (int)(i % a.Cs);
    const long r = i / a.Cs;
    const int t = (int)(r % a.ntaps);
    const long n = r / a.ntaps;
    const long g = blockIdx.z;
    ((T *)a.out)[g * total + i] = c < a.Cr ? ((const T *)a.w)[g * a.w_gstep + n * a.sn + a.tap_off[t] + c * a.sc] : (T)0.f;
}

// The gather for the small filters of many layers (a launch of its own takes each of them 2.7 us, nearly all of it the launch).
constexpr int kPackMany = 40;
struct PackMany {
    PackItem e[kPackMany];
    int count;
};
static_assert(sizeof(PackMany) <= 4096, "kernel arguments");
template <typename T> __global__ __launch_bounds__(256) void pack_many_kernel(const PackMany m)
{
    int k = 0;
    while (k + 1 < m.count && (int)blockIdx.x >= m.e[k + 1].first_block) ++k;
    const PackItem &a = m.e[k];
    const int i = ((int)blockIdx.x - a.first_block) * 256 + (int)threadIdx.x;
    if (i >= a.Nn * a.ntaps * a.Cs) return;
    const int r = i / a.Cs, c = i - r * a.Cs, n = r / a.ntaps, t = r - n * a.ntaps;
    ((T *)a.out)[i] = ((const T *)a.w)[n * a.sn + a.tap_off[t] + c * a.sc];
}

// The same where n runs along the source (sn = 1: backward-data of a KRSC filter), a transposition of every tap's [c][n] matrix: tiles
// of 64 c x 64 n (fp32: 32 n) through LDS with 16-byte accesses on both sides.  The gather above fetches a line for each element that
// a lane stores, 256 lines per block in flight: 512x512x9 bf16, 4.7 MB each way, 13.2 us there, 5.3 here.  Below 32 x 32
// channels most of a tile would be idle.  Rows of the tile are two bytes (fp32: four) times an odd number of banks apart.
template <typename T> __global__ __launch_bounds__(256) void pack_tiles_kernel(const PackMulti m)
{
    constexpr int VEC = 16 / (int)sizeof(T), TN = 8 * VEC, TC = 64, LD = TN + 4 / (int)sizeof(T);
    typedef T Vec __attribute__((ext_vector_type(VEC)));
    __shared__ T tile[TC][LD];
    const PackArgs &a = m.e[blockIdx.y];
    const int tn = (a.Nn + TN - 1) / TN, tc = (a.Cs + TC - 1) / TC;
    int b = blockIdx.x;
    const int t = b / (tn * tc);
    if (t >= a.ntaps) return;
    b -= t * tn * tc;
    const int n0 = b % tn * TN, c0 = b / tn * TC;
    const T *w = (const T *)a.w + (long)blockIdx.z * a.w_gstep + a.tap_off[t];
    T *out = (T *)a.out + ((long)blockIdx.z * a.Nn * a.ntaps + t) * a.Cs;
    for (int i = threadIdx.x; i < TC * 8; i += 256) {
        const int c = i >> 3, v = (i & 7) * VEC;
        Vec x = {};
        if (c0 + c < a.Cr && n0 + v < a.Nn) x = *(const Vec *)(w + (c0 + c) * a.sc + n0 + v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) tile[c][v + e] = x[e];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < TN * (TC / VEC); i += 256) {
        const int v = i % (TC / VEC) * VEC, n = i / (TC / VEC);
        if (c0 + v >= a.Cs || n0 + n >= a.Nn) continue;
        Vec x;
#pragma unroll
        for (int e = 0; e < VEC; ++e) x[e] = tile[v + e][n];
        *(Vec *)(out + (long)(n0 + n) * a.ntaps * a.Cs + c0 + v) = x;
    }
}

// Rows of `in` bytes -> rows of `out` bytes (a multiple of 16), the rest zeros: an activation whose channel count is not a
// whole number of 16-byte vectors, for the kernels that read such vectors.  A thread writes one vector from units of UNIT
// bytes (rows begin on multiples of UNIT).  Bound by memory and the launch: 5 MB of bf16 rows of 100 channels in 4.7 us.
template <typename U>
__global__ __launch_bounds__(256) void pad_rows_kernel(const U *__restrict__ src, u32x4 *__restrict__ dst, unsigned nvec, unsigned vpr, int units)
{
    constexpr int PER = 16 / (int)sizeof(U);
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < nvec; i += gridDim.x * 256) {
        const unsigned row = i / vpr;
        const int u0 = (int)(i - row * vpr) * PER;
        const U *p = src + (size_t)row * units + u0;
        union { U u[PER]; u32x4 v; } r;
#pragma unroll
        for (int e = 0; e < PER; ++e) r.u[e] = u0 + e < units ? p[e] : U{};
        dst[i] = r.v;
    }
}

// Zero the pixels (i*osh + oa, j*osw + ob), i < Mi, j < Mj, of every image of an NHWC tensor: the cells
// of a strided backward-data result that no filter tap reaches.  `unit` = bytes written per thread.
__global__ __launch_bounds__(256) void zero_class_kernel(unsigned char *__restrict__ out, long total, int Mi, int Mj, int Ho,
                                                         int Wo, int osh, int oa, int osw, int ob, int pix_bytes,
                                                         int unit)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int upp = pix_bytes / unit;            // units per pixel
    const int u = (int)(i % upp);
    long r = i / upp;
    const int j = (int)(r % Mj); r /= Mj;
    const int ii = (int)(r % Mi);
    const long img = r / Mi;
    unsigned char *p = out + ((img * Ho + (ii * osh + oa)) * Wo + (j * osw + ob)) * (long)pix_bytes + (long)u * unit;
    if (unit == 16) *(f32x4 *)p = f32x4{0.f, 0.f, 0.f, 0.f};
    else if (unit == 4) *(float *)p = 0.f;
    else *(unsigned short *)p = 0;
}

template <typename T>
int transpose_typed(const void *src, void *dst, int batch, int rows, int cols, int ldo, int accumulate, hipStream_t stream)
{
    dim3 grid(ceil_div(cols, 32), ceil_div(ldo, 32), batch);
    hipLaunchKernelGGL((transpose_kernel<T>), grid, dim3(256), 0, stream, (const T *)src, (T *)dst, rows, cols,
                       ldo, accumulate);
    return check_launch();
}

}  // namespace

int launch_nchw_to_nhwc(int dtype, const void *src, void *dst, int N, int C, int H, int W, int Cp, hipStream_t stream)
{
    if (dtype == NSK_BF16) return transpose_typed<bf16_t>(src, dst, N, C, H * W, Cp, 0, stream);
    return transpose_typed<float>(src, dst, N, C, H * W, Cp, 0, stream);
}

int launch_pad_channels(int dtype, const void *src, void *dst, long rows, int C, int Cp, hipStream_t stream)
{
    const unsigned es = (unsigned)elem_size(dtype), vpr = (unsigned)Cp * es / 16, bytes = (unsigned)C * es;
    const unsigned nvec = (unsigned)(rows * vpr);      // (below 2^32 bytes: activations are)
    const dim3 grid(nvec / 256 + 1 < 256 * 16 ? nvec / 256 + 1 : 256 * 16);
    if (bytes % 8 == 0)
        hipLaunchKernelGGL(pad_rows_kernel<unsigned long long>, grid, dim3(256), 0, stream, (const unsigned long long *)src, (u32x4 *)dst, nvec, vpr, (int)(bytes / 8));
    else if (bytes % 4 == 0)
        hipLaunchKernelGGL(pad_rows_kernel<unsigned>, grid, dim3(256), 0, stream, (const unsigned *)src, (u32x4 *)dst, nvec, vpr, (int)(bytes / 4));
    else
        hipLaunchKernelGGL(pad_rows_kernel<unsigned short>, grid, dim3(256), 0, stream, (const unsigned short *)src, (u32x4 *)dst, nvec, vpr, (int)(bytes / 2));
    return check_launch();
}

int launch_nhwc_to_nchw(int dtype, const void *src, void *dst, int N, int C, int H, int W, int accumulate,
                        hipStream_t stream)
{
    if (dtype == NSK_BF16) return transpose_typed<bf16_t>(src, dst, N, H * W, C, H * W, accumulate, stream);
    return transpose_typed<float>(src, dst, N, H * W, C, H * W, accumulate, stream);
}

int launch_zero_class(int dtype, void *out, int Nimg, int Ho, int Wo, int Co, int Mi, int Mj, int osh, int oa, int osw,
                      int ob, hipStream_t stream)
{
    const int pix_bytes = Co * (int)elem_size(dtype);
    const int unit = pix_bytes % 16 == 0 ? 16 : (pix_bytes % 4 == 0 ? 4 : 2);
    const long total = (long)Nimg * Mi * Mj * (pix_bytes / unit);
    if (total == 0) return NSK_OK;
    hipLaunchKernelGGL(zero_class_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, (unsigned char *)out,
                       total, Mi, Mj, Ho, Wo, osh, oa, osw, ob, pix_bytes, unit);
    return check_launch();
}

int launch_pack_filters_grouped(int dtype, int count, const void *w, void *const *out, int Nn, const int *ntaps, int Cs, int Cr,
                                long sn, long sc, const int (*tap_off_host)[kMaxTaps], int groups, long w_gstep,
                                hipStream_t stream)
{
    if (count < 1 || count > kPackMulti || groups < 1 || groups > 65535) return NSK_ERR_BAD_DESC;
    PackMulti m{};
    long most = 0;
    for (int k = 0; k < count; ++k) {
        PackArgs &a = m.e[k];
        a.w = w;
        a.out = out[k];
        a.Nn = Nn;
        a.ntaps = ntaps[k];
        a.Cs = Cs;
        a.Cr = Cr;
        a.sn = sn;
        a.sc = sc;
        a.w_gstep = w_gstep;
        for (int t = 0; t < kMaxTaps; ++t) a.tap_off[t] = t < ntaps[k] ? tap_off_host[k][t] : 0;
        const long total = (long)Nn * ntaps[k] * Cs;
        if (total > most) most = total;
    }
    if (most == 0) return NSK_OK;
    // Whole vectors on both sides; from 140000 elements on, below the gather is as fast or faster (backward-data of 8 images of 8x8 with its
    // pack, gather / tiles, us: 64 -> 64 3x3 7.8 / 8.2, 512 -> 256 1x1 7.7 / 8.0, 128 -> 128 3x3 12.4 / 11.8, 512 -> 512 1x1 9.3 / 8.8)
    const long vec = dtype == NSK_BF16 ? 8 : 4;
    bool tiles = sn == 1 && most * groups >= 140000 && Nn >= 32 && Cs >= 32 && Nn % vec == 0 && Cs % vec == 0 && sc % vec == 0 && w_gstep % vec == 0 && ((uintptr_t)w & 15) == 0;
    for (int k = 0; k < count; ++k) {
        tiles = tiles && ((uintptr_t)out[k] & 15) == 0;
        for (int t = 0; t < ntaps[k]; ++t) tiles = tiles && tap_off_host[k][t] % vec == 0;
    }
    if (tiles) {
        int taps = 0;
        for (int k = 0; k < count; ++k) taps = ntaps[k] > taps ? ntaps[k] : taps;
        dim3 grid((unsigned)(taps * ceil_div(Nn, 8 * (int)vec) * ceil_div(Cs, 64)), (unsigned)count, (unsigned)groups);
        if (dtype == NSK_BF16)
            hipLaunchKernelGGL((pack_tiles_kernel<bf16_t>), grid, dim3(256), 0, stream, m);
        else
            hipLaunchKernelGGL((pack_tiles_kernel<float>), grid, dim3(256), 0, stream, m);
        return check_launch();
    }
    dim3 grid((unsigned)((most + 255) / 256), (unsigned)count, (unsigned)groups);
    if (dtype == NSK_BF16)
        hipLaunchKernelGGL((pack_filter_kernel<bf16_t>), grid, dim3(256), 0, stream, m);
    else
        hipLaunchKernelGGL((pack_filter_kernel<float>), grid, dim3(256), 0, stream, m);
    return check_launch();
}

int launch_pack_many(int dtype, PackItem *items, int count, hipStream_t stream)
{
    for (int at = 0; at < count; at += kPackMany) {
        PackMany m{};
        m.count = count - at < kPackMany ? count - at : kPackMany;
        int blocks = 0;
        for (int k = 0; k < m.count; ++k) {
            items[at + k].first_block = blocks;
            blocks += ceil_div(items[at + k].Nn * items[at + k].ntaps * items[at + k].Cs, 256);
            m.e[k] = items[at + k];
        }
        if (blocks == 0) continue;
        if (dtype == NSK_BF16)
            hipLaunchKernelGGL((pack_many_kernel<bf16_t>), dim3((unsigned)blocks), dim3(256), 0, stream, m);
        else
            hipLaunchKernelGGL((pack_many_kernel<float>), dim3((unsigned)blocks), dim3(256), 0, stream, m);
        const int rc = check_launch();
        if (rc != NSK_OK) return rc;
    }
    return NSK_OK;
}

int launch_pack_filter(int dtype, const void *w, void *out, int Nn, int ntaps, int Cs, int Cr, long sn, long sc,
                       const int *tap_off_host, hipStream_t stream)
{
    int taps[1][kMaxTaps];
    for (int t = 0; t < kMaxTaps; ++t) taps[0][t] = t < ntaps ? tap_off_host[t] : 0;
    void *outs[1] = {out};
    return launch_pack_filters_grouped(dtype, 1, w, outs, Nn, &ntaps, Cs, Cr, sn, sc, taps, 1, 0L, stream);
}

}  // namespace nsk
