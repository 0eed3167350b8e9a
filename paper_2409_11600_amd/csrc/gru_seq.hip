// All time steps of the GRU in one launch per direction, for few samples and hidden sizes up to 256.
//
// What bounds the step-by-step form: 2T dependent launches of 5.5-7 us each (a launch, an L2 round trip for the operands, a
// store) and as many calls from the host.  But a sample's state depends on that sample alone: here a block owns one sample
// and runs all T steps by itself, so nothing is exchanged between blocks and nothing is launched in between.  What has to
// be at hand in every step is the whole recurrent weight (3*H*H values: 786 KB in fp32 at H = 256, more than the 512 KB of
// registers and 160 KB of LDS of a CU): a thread keeps most of its part in registers for all T steps, some of it lies in
// LDS, and in fp32 above H = 192 the rest is read from L2 again in every step, while the resident part is multiplied.
//
// Work inside a block of 512 threads: eight neighbouring lanes q share a hidden unit's dot products (lane q takes the
// columns 4*(q + 8*m) ..), 64 groups of lanes hold the units slot, slot + 64, ...; the lane sums run over the eight lanes
// in a fixed order, then lane q goes on with the gates of unit slot + 64*q.  The state (forward) or the gate gradients
// (backward) go through LDS, double-buffered: one barrier per step.
//
// Measured, us for T = 200 steps (step launches -> this kernel, forward / backward): fp32, 50 samples, H = 256: 973 / 1255 ->
// 705 / 619 (and 2.4 ms of host calls gone); H = 192: 859 / 1142 -> 363 / 293; H = 64: 627 / 688 -> 147 / 134; bf16, H = 256:
// 1065 / 1218 -> 395 / 322; fp32, 200 samples, H = 256: 2843 / 3435 -> 805 / 705.  A training step of the fp32 model with 50
// samples, H = 256, T = 200: 5.4 -> 1.8 ms.  At H = 256 in fp32 a step is bound by the 5/12 of the weight that a block
// reads from L2 (328 KB per step); below, by the LDS reads, the lane sums and the chain of the gates.
#include <math.h>

#include "nsk_internal.h"

namespace nsk {
namespace {

bool unaligned16(const void *p) { return ((uintptr_t)p & 15) != 0; }

__device__ inline float sigmoidf(float a) { return 1.f / (1.f + expf(-a)); }

typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));

template <typename T> struct SeqT;
template <> struct SeqT<float> {
    typedef f32x4 V;
    static __device__ inline float mac(float a, V w, V v)
    {
        float t = w[0] * v[0];      // four products at a time: chains of 4 and 8 roundings, not one of 32
#pragma unroll
        for (int e = 1; e < 4; ++e) t = fmaf(w[e], v[e], t);
        return a + t;
    }
    static __device__ inline V fetch(__amdgpu_buffer_rsrc_t r, unsigned at) { return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0)); }
};
template <> struct SeqT<bf16_t> {
    typedef bf16x4 V;
    static __device__ inline float mac(float a, V w, V v)
    {
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 0, 1), __builtin_shufflevector(v, v, 0, 1), a, false);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 2, 3), __builtin_shufflevector(v, v, 2, 3), a, false);
    }
    static __device__ inline V fetch(__amdgpu_buffer_rsrc_t r, unsigned at) { return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, (int)at, 0, 0)); }
};

constexpr int GQ_THREADS = 512;

struct GruSeqArgs {
    const void *gi, *w, *saved_in, *dh_top;      // w: W_hh [3H][H] forward, its transpose [H][3H] backward
    const float *b_ih, *b_hh;
    void *h, *saved, *dgi, *dgh;
    int T, N, H;
};

// IU = units per thread, M = 4-column pieces per lane and gate; of the 3*IU (unit, gate) parts RS stay in registers, LS in LDS
template <typename T, bool BWD, int IU, int M, int RS, int LS>
__global__ __launch_bounds__(GQ_THREADS) void gru_seq_kernel(const GruSeqArgs a)
{
    typedef SeqT<T> ST;
    typedef typename ST::V V;
    constexpr int S = 3 * IU, SS = S - RS - LS, HP = 32 * M, NV = BWD ? 3 : 1;
    static_assert(SS >= 0, "parts");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *const vec = (T *)smem;                                   // [2][NV][HP]: what the step multiplies
    V *const lw = (V *)(smem + 2 * NV * HP * sizeof(T));        // [LS][M][512]
    const int tid = threadIdx.x, q = tid & 7, slot = tid >> 3, n = blockIdx.x, H = a.H, N = a.N;

    // part p = (unit slot + 64*(p/3), gate p%3): byte offset of its row of this thread's columns; columns past H read zeros
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.w, 0, (unsigned)(3 * H * H * (int)sizeof(T)), 0x00020000);
    auto row = [&](int p) -> unsigned {
        const int u = min(slot + 64 * (p / 3), H - 1), g = p % 3;
        return (unsigned)((BWD ? u * 3 * H + g * H : (g * H + u) * H) + 4 * q) * (unsigned)sizeof(T);
    };
    auto column = [&](int m) { return 4 * (q + 8 * m); };
    auto load = [&](unsigned r, int m) -> V {
        const unsigned at = r + (unsigned)(32 * m * (int)sizeof(T));
        if (32 * m + 32 <= 64 * (IU - 1)) return ST::fetch(w_rsrc, at);     // (H > 64*(IU - 1))
        return ST::fetch(w_rsrc, column(m) < H ? at : ~0u);
    };
    V wr[RS][M];
#pragma unroll
    for (int p = 0; p < RS; ++p)
#pragma unroll
        for (int m = 0; m < M; ++m) wr[p][m] = load(row(p), m);
#pragma unroll
    for (int p = 0; p < LS; ++p)
#pragma unroll
        for (int m = 0; m < M; ++m) lw[(p * M + m) * GQ_THREADS + tid] = load(row(RS + p), m);
    // The parts that fit nowhere: one piece of each at a time.  The next piece is requested as soon as the one before has been
    // used, so it is on its way while the resident parts are multiplied; the first piece of a step comes during the gates
    // of the step before.
    unsigned rs[SS > 0 ? SS : 1];
    V sw[SS > 0 ? SS : 1];
#pragma unroll
    for (int p = 0; p < SS; ++p) {
        rs[p] = row(RS + LS + p);
        sw[p] = load(rs[p], 0);
    }
    for (int i = tid; i < 2 * NV * HP; i += GQ_THREADS) vec[i] = (T)0.f;
    __syncthreads();

    // this lane's unit in the elementwise part
    const int u = slot + 64 * q;
    const bool mine = q < IU && u < H;
    const int ue = mine ? u : 0;
    const long NH = (long)N * H, at = (long)n * H + ue;
    float br = 0.f, bz = 0.f, bin = 0.f, bhn = 0.f, state = 0.f;   // state: h (forward), the direct part of dh (backward)
    if constexpr (!BWD) {
        br = a.b_ih[ue] + a.b_hh[ue];
        bz = a.b_ih[H + ue] + a.b_hh[H + ue];
        bin = a.b_ih[2 * H + ue];
        bhn = a.b_hh[2 * H + ue];
        state = (float)((const T *)a.h)[at];
        if (mine) vec[u] = (T)state;
        __syncthreads();
    } else {
        state = (float)((const T *)a.dh_top)[at];
    }

    for (int step = 0; step < a.T; ++step) {
        const int t = BWD ? a.T - 1 - step : step, buf = step & 1;
        // the elementwise operands are requested before the products
        float e0, e1, e2, e3 = 0.f, e4 = 0.f;
        if constexpr (!BWD) {
            const T *gi = (const T *)a.gi + (long)t * 3 * NH + (long)n * 3 * H + ue;
            e0 = (float)gi[0];
            e1 = (float)gi[H];
            e2 = (float)gi[2 * H];
        } else {
            const T *sv = (const T *)a.saved_in + (long)t * 4 * NH + (long)n * 4 * H + ue;
            e0 = (float)sv[0];
            e1 = (float)sv[H];
            e2 = (float)sv[2 * H];
            e3 = (float)sv[3 * H];
            e4 = (float)((const T *)a.h)[(long)t * NH + at];
        }
        float acc[S];
#pragma unroll
        for (int p = 0; p < S; ++p) acc[p] = 0.f;
        {
            const T *v0 = vec + buf * NV * HP;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                V v[NV];
#pragma unroll
                for (int g = 0; g < NV; ++g) v[g] = *(const V *)(v0 + g * HP + column(m));
#pragma unroll
                for (int p = 0; p < SS; ++p) {
                    acc[RS + LS + p] = ST::mac(acc[RS + LS + p], sw[p], v[BWD ? (RS + LS + p) % 3 : 0]);
                    sw[p] = load(rs[p], (m + 1) % M);
                }
#pragma unroll
                for (int p = 0; p < RS; ++p) acc[p] = ST::mac(acc[p], wr[p][m], v[BWD ? p % 3 : 0]);
#pragma unroll
                for (int p = 0; p < LS; ++p) acc[RS + p] = ST::mac(acc[RS + p], lw[(p * M + m) * GQ_THREADS + tid], v[BWD ? (RS + p) % 3 : 0]);
                __builtin_amdgcn_sched_barrier(0);     // (or every piece of the step is fetched ahead, into scratch)
            }
        }
        if constexpr (BWD) {
#pragma unroll
            for (int i = 0; i < IU; ++i) {
                acc[i] = (acc[3 * i] + acc[3 * i + 1]) + acc[3 * i + 2];
                acc[i] = step > 0 ? acc[i] : 0.f;    // (no step comes after the last one)
            }
        }
        constexpr int R = BWD ? IU : S;
#pragma unroll
        for (int p = 0; p < R; ++p) {
#pragma unroll
            for (int o = 1; o < 8; o <<= 1) acc[p] += __shfl_xor(acc[p], o, 64);
        }
        T *vn = vec + (buf ^ 1) * NV * HP;
        if constexpr (!BWD) {
            float gr = acc[0], gz = acc[1], gn = acc[2];
#pragma unroll
            for (int i = 1; i < IU; ++i) {
                gr = q == i ? acc[3 * i] : gr;
                gz = q == i ? acc[3 * i + 1] : gz;
                gn = q == i ? acc[3 * i + 2] : gn;
            }
            if (mine) {
                const float r = sigmoidf(e0 + gr + br);
                const float z = sigmoidf(e1 + gz + bz);
                const float qq = gn + bhn;
                const float c = tanhf(e2 + bin + r * qq);
                const T hn = (T)((1.f - z) * c + z * state);
                state = (float)hn;
                vn[u] = hn;
                ((T *)a.h)[(long)(t + 1) * NH + at] = hn;
                T *sv = (T *)a.saved + (long)t * 4 * NH + (long)n * 4 * H + u;
                sv[0] = (T)r;
                sv[H] = (T)z;
                sv[2 * H] = (T)c;
                sv[3 * H] = (T)qq;
            }
        } else {
            // (the sums of the units i >= 1 lie at acc[i])
            float dh = acc[0];
#pragma unroll
            for (int i = 1; i < IU; ++i) dh = q == i ? acc[i] : dh;
            if (mine) {
                dh += state;
                const float r = e0, z = e1, c = e2, qq = e3;
                const float da_n = dh * (1.f - z) * (1.f - c * c);
                const float da_z = dh * (e4 - c) * z * (1.f - z);
                const float da_r = da_n * qq * r * (1.f - r);
                state = (float)(T)(dh * z);
                const T tr = (T)da_r, tz = (T)da_z, tn = (T)(da_n * r);
                vn[u] = tr;
                vn[HP + u] = tz;
                vn[2 * HP + u] = tn;
                const long g0 = (long)t * 3 * NH + (long)n * 3 * H + u;
                T *dgi = (T *)a.dgi + g0, *dgh = (T *)a.dgh + g0;
                dgi[0] = tr;
                dgi[H] = tz;
                dgi[2 * H] = (T)da_n;
                dgh[0] = tr;
                dgh[H] = tz;
                dgh[2 * H] = tn;
            }
        }
        lds_barrier();
    }
}

template <typename T, bool BWD, int IU, int M, int RS, int LS> int launch(const GruSeqArgs &a, hipStream_t stream)
{
    const size_t smem = 2 * (BWD ? 3 : 1) * 32 * M * sizeof(T) + (size_t)LS * M * GQ_THREADS * 4 * sizeof(T);
    static std::atomic<unsigned long long> done{0};
    if (smem > 64 * 1024) {
        const int rc = allow_lds((const void *)gru_seq_kernel<T, BWD, IU, M, RS, LS>, smem, done);
        if (rc != NSK_OK) return rc;
    }
    hipLaunchKernelGGL((gru_seq_kernel<T, BWD, IU, M, RS, LS>), dim3(a.N), dim3(GQ_THREADS), smem, stream, a);
    return check_launch();
}

// The split of the parts is what the register file takes without spilling (512 threads: 256 registers each), the rest in LDS.
// fp32 at H > 192, forward / backward in us: 5 parts in registers 705 / 619, 4 parts 775 / 691, 3 parts 893 / 784; 6 spill:
// 807 / 862.
template <bool BWD> int dispatch(int dtype, const GruSeqArgs &a, hipStream_t stream)
{
    const int m = (a.H + 63) / 64;
    if (dtype == NSK_BF16) {
        switch (m) {
        case 1: return launch<bf16_t, BWD, 1, 2, 3, 0>(a, stream);
        case 2: return launch<bf16_t, BWD, 2, 4, 6, 0>(a, stream);
        case 3: return launch<bf16_t, BWD, 3, 6, 9, 0>(a, stream);
        default: return launch<bf16_t, BWD, 4, 8, 9, 3>(a, stream);
        }
    }
    switch (m) {
    case 1: return launch<float, BWD, 1, 2, 3, 0>(a, stream);
    case 2: return launch<float, BWD, 2, 4, 6, 0>(a, stream);
    case 3: return launch<float, BWD, 3, 6, 7, 2>(a, stream);
    default: return launch<float, BWD, 4, 8, 5, 2>(a, stream);
    }
}

// One block holds a CU for the whole sequence.  Above 256 units a block would read nearly all of the weight again in every step,
// which the step launches spread over the chip; N is at most the 256 that the step calls take, so one wave of blocks.
bool seq_kernel_takes(int H) { return H <= 256; }

}  // namespace
}  // namespace nsk

using namespace nsk;

extern "C" {

int nsk_gru_seq_fwd(int dtype, int T, int N, int H, const void *gi, const void *w_hh, const float *b_ih, const float *b_hh,
                    void *h, void *saved, void *stream)
{
    if (T <= 0 || N <= 0 || H <= 0 || (dtype != NSK_F32 && dtype != NSK_BF16)) return NSK_ERR_BAD_DESC;
    if (!gi || !w_hh || !b_ih || !b_hh || !h || !saved) return NSK_ERR_NULL;
    const size_t es = dtype == NSK_BF16 ? 2 : 4, step = (size_t)N * H * es;
    if (unaligned16(gi) || unaligned16(w_hh) || unaligned16(b_ih) || unaligned16(b_hh) || unaligned16(h) || unaligned16(saved) ||
        step % 16 != 0)
        return NSK_ERR_ALIGNMENT;
    if (!nsk_gru_step_supported(N, H)) return NSK_ERR_UNSUPPORTED;
    if (seq_kernel_takes(H)) {
        GruSeqArgs a{};
        a.gi = gi; a.w = w_hh; a.b_ih = b_ih; a.b_hh = b_hh; a.h = h; a.saved = saved;
        a.T = T; a.N = N; a.H = H;
        return dispatch<false>(dtype, a, (hipStream_t)stream);
    }
    for (int t = 0; t < T; ++t) {
        char *hp = (char *)h + (size_t)t * step;
        const int rc = nsk_gru_step_fwd(dtype, N, H, (const char *)gi + (size_t)t * 3 * step, w_hh, b_ih, b_hh, hp, hp + step,
                                        (char *)saved + (size_t)t * 4 * step, stream);
        if (rc != NSK_OK) return rc;
    }
    return NSK_OK;
}

int nsk_gru_seq_bwd(int dtype, int T, int N, int H, const void *saved, const void *h, const void *dh_top, const void *w_hh_t,
                    void *dgi, void *dgh, void *dh_scratch, void *stream)
{
    if (T <= 0 || N <= 0 || H <= 0 || (dtype != NSK_F32 && dtype != NSK_BF16)) return NSK_ERR_BAD_DESC;
    if (!saved || !h || !dh_top || !w_hh_t || !dgi || !dgh || !dh_scratch) return NSK_ERR_NULL;
    const size_t es = dtype == NSK_BF16 ? 2 : 4, step = (size_t)N * H * es;
    if (unaligned16(saved) || unaligned16(h) || unaligned16(dh_top) || unaligned16(w_hh_t) || unaligned16(dgi) || unaligned16(dgh) ||
        unaligned16(dh_scratch) || step % 16 != 0)
        return NSK_ERR_ALIGNMENT;
    if (!nsk_gru_step_supported(N, H)) return NSK_ERR_UNSUPPORTED;
    if (seq_kernel_takes(H)) {
        GruSeqArgs a{};
        a.saved_in = saved; a.h = (void *)h; a.dh_top = dh_top; a.w = w_hh_t; a.dgi = dgi; a.dgh = dgh;
        a.T = T; a.N = N; a.H = H;
        return dispatch<true>(dtype, a, (hipStream_t)stream);
    }
    for (int t = T - 1; t >= 0; --t) {
        const bool last = t == T - 1;
        char *direct = (char *)dh_scratch + (size_t)(t & 1) * step, *next = (char *)dh_scratch + (size_t)((t & 1) ^ 1) * step;
        char *g = (char *)dgh + (size_t)t * 3 * step;
        const int rc = nsk_gru_step_bwd(dtype, N, H, (const char *)saved + (size_t)t * 4 * step, (const char *)h + (size_t)t * step,
                                        last ? dh_top : nullptr, last ? nullptr : next, last ? nullptr : g + 3 * step, w_hh_t,
                                        (char *)dgi + (size_t)t * 3 * step, g, direct, stream);
        if (rc != NSK_OK) return rc;
    }
    return NSK_OK;
}

}  // extern "C"
