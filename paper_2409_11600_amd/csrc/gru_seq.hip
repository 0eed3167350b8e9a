// All time steps of the GRU in one launch per direction, for few samples and hidden sizes up to 256.
//
// What bounds the step-by-step form: 2T dependent launches of 5.5-7 us each (a launch, an L2 round trip for the operands, a
// store) and as many calls from the host.  But a sample's state depends on that sample alone: here G blocks own one sample
// and run all T steps by themselves.  What has to be at hand in every step is the whole recurrent weight (3*H*H values: 786 KB
// in fp32 at H = 256, more than the 512 KB of registers and 160 KB of LDS of a CU).
//
// G = 1: a block has the sample to itself and nothing is exchanged.  A thread keeps most of its part of the weight in registers
// for all T steps, some of it lies in LDS, and in fp32 above H = 192 the rest is read from L2 again in every step, while the
// resident part is multiplied.
//
// G = 2 or 4 (few samples): each block owns H/G of the hidden units, so its part of the weight stays on the CU and a step's
// products take 1/G of the time; what it pays is an exchange per step.  The exchange goes through the output itself (h forward,
// dgh backward): a fill launch puts a NaN that no step stores in front of it, a block's gate lanes store their units with
// atomics, and a wavefront of its own per vector polls the others' values until none of them is that NaN, so value
// and flag arrive together (a store of agent scope and the load that sees it take 0.45 us on one XCD, 0.63 us across; a store into the L2 of
// the XCD and an agent-scope load there 0.22 us).  The members of a group are blocks b, b + 8, ..: one XCD when blocks go round the eight.
// They tell each other theirs at the first steps, and a block whose readers all share its XCD stores into the L2 from then on; where
// that did not reach a reader, it would give up like any other.  The pollers are wavefronts of their own because a
// wavefront's loads return in order: behind the elementwise operands, which come from HBM, every poll would wait for those.
// Waiting ends: members of a group are dispatched one after the other and hold no more CUs than the XCD has (split_of), and whole
// groups wait for nobody else.  So of each launch at most one group an XCD, G - 1 blocks, waits for a block that has no CU yet: ten launches
// at a time on one card leave CUs free for those.  With more, or where others hold the CUs for long, a poller that has seen kPolls polls
// fail gives up: its block goes on with what it has, and in the end puts the mark back into that sample's last row.  A launch of the
// G = 1 kernel behind looks at the last rows and runs the samples that have the mark, from their first step: same bits, so
// the call is right in any case, and such a sample costs that wait and the time without a split.  (Ending such a block at once, by a
// word in LDS that every step looks at, cost the two-block kernel 28 bytes of scratch a thread: 57 / 59 -> 76 / 72 us for 20 steps.)
//
// Work inside a block of 512 (32 units: 256) multiplying threads: eight neighbouring lanes q share a hidden unit's dot products
// (lane q takes the columns 4*(q + 8*m) ..), 64 (32) groups of lanes hold the units slot, slot + 64, ...; the lane sums run over
// the eight lanes in a fixed order, then lane q goes on with the gates of unit slot + 64*q.  The state (forward) or the gate
// gradients (backward) go through LDS, double-buffered: one barrier per step.
//
// Measured, us for T = 200 steps (step launches -> this kernel, forward / backward): fp32, 50 samples, H = 256: 973 / 1255
// -> 277 / 314 (one block per sample 574 / 594; 303 / 336 with every exchange through memory); H = 192: 859 / 1142 -> 282 / 277; H = 64:
// 627 / 688 -> 111 / 113; bf16, H = 256: 1065 / 1218 -> 232 / 264.  A split step of 1.4 - 1.6 us is 0.5 us of exchange, 0.35 us of products and the chain of sums and gates; without a
// split it is that chain (0.5 us), the products and, at H = 256, the part of the weight that comes from L2.
#include <math.h>

#include <algorithm>

#include "nsk_internal.h"

namespace nsk {
namespace {

bool unaligned16(const void *p) { return ((uintptr_t)p & 15) != 0; }

// Gate functions, written for a chain of few dependent instructions (a step is one chain; the library's take 1.5 times as many):
// exp as the hardware's 2^t with the rounding of t = x*log2(e) put back as a factor, a reciprocal of 1 + e with one Newton step, tanh as
// 1 - 2/(e^2x + 1) and, below 0.75 where that cancels, as an odd polynomial (least squares on Chebyshev nodes, relative error 7e-9).  Arguments
// of exp are held at +-88, where it stays finite; NaN goes through.  Mean errors of r, z, tanh and h against 64 bits over five sizes:
// 3.1, 3.1, 4.3, 7.4e-8 (with the library's functions 4.2, 4.2, 4.3, 8.1e-8).
__device__ inline float exp_to88(float x)
{
    x = x > 88.f ? 88.f : x < -88.f ? -88.f : x;
    const float t = x * 1.44269502f;
    const float lo = fmaf(x, 1.44269502f, -t) + x * 1.92596303e-8f;
    const float e = __builtin_amdgcn_exp2f(t);
    return fmaf(e, lo * 0.693147182f, e);
}
// 1 / (1 + e), the rounding of 1 + e put back in the Newton step
__device__ inline float reciprocal1p(float e)
{
    const float d = 1.f + e, r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(d - 1.f - e, r, fmaf(-d, r, 1.f)), r, r);
}
__device__ inline float gate_sigmoid(float a) { return reciprocal1p(exp_to88(-a)); }
__device__ inline float gate_tanh(float a)
{
    const float x = fabsf(a), z = x * x;
    const float big = fmaf(-2.f, reciprocal1p(exp_to88(2.f * x)), 1.f);
    float p = fmaf(0.00191453542f, z, -0.007940921f);
    p = fmaf(p, z, 0.0216188431f);
    p = fmaf(p, z, -0.0539365672f);
    p = fmaf(p, z, 0.13333185f);
    p = fmaf(p, z, -0.333333313f);
    const float y = x < 0.75f ? fmaf(x * z, p, x) : big;
    return copysignf(y, a);
}

typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));

template <typename T> struct SeqT;
template <> struct SeqT<float> {
    typedef f32x4 V;
    typedef unsigned U;
    // FOUR: four products at a time, chains of 4 and 8 roundings and not one of 32, for a fifth instruction
    template <bool FOUR> static __device__ inline float mac(float a, V w, V v)
    {
        float t = FOUR ? w[0] * v[0] : fmaf(w[0], v[0], a);
#pragma unroll
        for (int e = 1; e < 4; ++e) t = fmaf(w[e], v[e], t);
        return FOUR ? a + t : t;
    }
    static __device__ inline V fetch(__amdgpu_buffer_rsrc_t r, unsigned at) { return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0)); }
};
template <> struct SeqT<bf16_t> {
    typedef bf16x4 V;
    typedef unsigned short U;
    template <bool FOUR> static __device__ inline float mac(float a, V w, V v)
    {
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 0, 1), __builtin_shufflevector(v, v, 0, 1), a, false);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 2, 3), __builtin_shufflevector(v, v, 2, 3), a, false);
    }
    static __device__ inline V fetch(__amdgpu_buffer_rsrc_t r, unsigned at) { return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, (int)at, 0, 0)); }
};

constexpr unsigned kUnset = 0xffffffffu;      // a NaN in fp32 and, twice, in bf16; NaNs that a step stores are 0x7fc0(0000)
constexpr int kPolls = 1 << 20;               // failed polls of a wavefront before it gives up: about a second
// Polls cross the chip (650 ns there and back, whoever stores) and slow the stores that they wait for: a poll that comes too early
// costs a second one, four on their way at a time cost 487 / 690 us where one alone costs 371 / 466.  So a poller sleeps before
// its first poll of a step, in quarters of 64 clocks: 16 more after a first poll that failed, one less after every step
// (against it 6 and 1 whole units -2 / +30 us, eighths 40 and 1 +5 / -7 us but unsteady).  Polls of a group that shares an XCD end in its L2,
// and a poller there does not sleep (8 samples 256 / 270 us, with 8 quarters more after a failed poll 266 / 279).
constexpr int kSleepUp = 16, kSleepMost = 256;
constexpr int kNearSteps = 4;                 // shortest sequence whose blocks tell each other their XCD

// sum over the eight lanes of a group, in every lane: neighbours 1 and 2 away, then the mirrored lane of the other four
__device__ inline float sum8(float v)
{
    auto other = [](float x, auto ctl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctl)::value, 0xf, 0xf, true));
    };
    v += other(v, std::integral_constant<int, 0xb1>{});     // quad_perm 1,0,3,2
    v += other(v, std::integral_constant<int, 0x4e>{});     // quad_perm 2,3,0,1
    v += other(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
    return v;
}

// values that blocks exchange: loaded at agent scope, which passes the CU's own cache by, and stored at that scope, which goes to memory, or,
// where the group's blocks share an XCD (near), into the L2 that they share.  The language promises the latter to nobody outside the block
// that stores: near is for gfx950, whose CUs write their stores through to the L2 of their XCD, where an agent-scope load from the same XCD finds them.  A
// chip on which it did not would cost time, not results: the reader gives up after kPolls polls.
template <typename U> __device__ inline void publish_bits(U *p, U b, bool near)
{
    if (near)
        __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void publish(float *p, float v, bool near)
{
    publish_bits((unsigned *)p, v != v ? 0x7fc00000u : __builtin_bit_cast(unsigned, v), near);
}
__device__ inline void publish(bf16_t *p, bf16_t v, bool near)
{
    publish_bits((unsigned short *)p, (float)v != (float)v ? (unsigned short)0x7fc0 : __builtin_bit_cast(unsigned short, v), near);
}
// A block's XCD as a value that no step stores (a NaN of another payload), in its lowest 4 bits
template <typename U> __device__ inline U xcd_code()
{
    const unsigned xcd = __builtin_amdgcn_s_getreg(20 | 3 << 11);      // HW_REG_XCC_ID, bits 0..3
    return (U)((sizeof(U) == 4 ? 0x7fc1a500u : 0x7fd0u) | xcd);
}
typedef unsigned long long u64;
__device__ inline u64 seen(const void *p) { return __hip_atomic_load((const u64 *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ inline bool unset(u64 v)
{
    if (sizeof(T) == 4) return (unsigned)v == kUnset || (unsigned)(v >> 32) == kUnset;
    bool any = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) any |= ((v >> (16 * e)) & 0xffff) == 0xffff;
    return any;
}

struct GruSeqArgs {
    const void *gi, *w, *saved_in, *dh_top;      // w: W_hh [3H][H] forward, its transpose [H][3H] backward
    const float *b_ih, *b_hh;
    void *h, *saved, *dgi, *dgh;
    int T, N, H;
    int G, HU;       // blocks per sample and units per block (1 and H where a block has the sample to itself)
    int apart;       // blocks of a sample lie so many apart: 8, on one XCD (1, test hook: on XCDs of their own)
    int polls;       // failed polls of a wavefront before it gives up
    bool unfinished; // G = 1: only the samples whose last row still holds the mark
};

// IU = units per thread, M = 4-column pieces per lane and gate; of the 3*IU (unit, gate) parts RS stay in registers, LS in LDS;
// SLOTS = groups of eight lanes; SPLIT: a.G blocks per sample
template <typename T, bool BWD, int IU, int M, int RS, int LS, int SLOTS, bool SPLIT>
__global__ __launch_bounds__(8 * SLOTS + (SPLIT ? 64 * (BWD ? 3 : 1) : 0)) void gru_seq_kernel(const GruSeqArgs a)
{
    typedef SeqT<T> ST;
    typedef typename ST::V V;
    constexpr int S = 3 * IU, SS = S - RS - LS, HP = 32 * M, NV = BWD ? 3 : 1, MT = 8 * SLOTS;
    constexpr bool FOUR = !(BWD && M == 4);     // (the chain of 16 there is as long as it was; 128 units, 50 samples, 200 steps 199 -> 191 us)
    static_assert(SS >= 0, "parts");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *const vec = (T *)smem;                                   // [2][NV][HP]: what the step multiplies
    V *const lw = (V *)(smem + 2 * NV * HP * sizeof(T));        // [LS][M][MT]
    int *const near_lds = (int *)(lw + LS * M * MT);            // SPLIT: the group's blocks share an XCD
    const int tid = threadIdx.x, q = tid & 7, slot = tid >> 3, H = a.H, N = a.N;
    // SPLIT: groups of G blocks
    const int block = (int)blockIdx.x, n = SPLIT ? block / (a.apart * a.G) * a.apart + block % a.apart : block;
    const int u0 = SPLIT ? block % (a.apart * a.G) / a.apart * a.HU : 0, u1 = SPLIT ? min(u0 + a.HU, H) : H;
    if (SPLIT && n >= N) return;
    const long NH = (long)N * H;
    if constexpr (!SPLIT) {
        if (a.unfinished) {
            const int words = (BWD ? 3 : 1) * H * (int)sizeof(T) / 8;      // of the row that the last step leaves
            const u64 *last = (const u64 *)(BWD ? (const T *)a.dgh + (long)n * 3 * H : (const T *)a.h + (long)a.T * NH + (long)n * H);
            bool un = false;
            for (int i = tid; i < words; i += MT) un |= unset<T>(last[i]);
            if (!__syncthreads_or(un)) return;
        }
    }

    if (SPLIT && tid >= MT) {
        // a polling wavefront: vector g of the step, four columns per lane
        const int g = (tid - MT) >> 6, c = 4 * (tid & 63);
        const bool live = c < H;
        int left = a.polls, wait = 0;
        bool gave_up = false, near = false;
        // The blocks' XCDs, by way of a place each that only the last step stores to: no block gets there before all have looked.
        typedef typename ST::U U;
        U *const codes = BWD ? (U *)a.dgi + (long)n * 3 * H : (U *)a.saved + (long)(a.T - 1) * 4 * NH + (long)n * 4 * H;
        const U code = xcd_code<U>();
        if (g == 0 && tid == MT) {
            *near_lds = 0;
            if (a.T >= kNearSteps) __hip_atomic_store(codes + u0, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (int step = 0; step < a.T; ++step) {
            if (step == 1 && g == 0 && a.T >= kNearSteps) {
                const U *other = codes + (tid & 63) % a.G * a.HU;
                U v = 0;
                for (int i = 0; i < 64 && __any((v & (U)~15u) != (code & (U)~15u)); ++i)
                    v = __hip_atomic_load(other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                near = !__any(v != code);
                if (tid == MT) *near_lds = near;
            }
            if (step == 2 && g > 0) near = *near_lds;
            if (step > 0 && live) {
                const int t = BWD ? a.T - step : step;          // the row that the step before this one has left
                const T *src = BWD ? (const T *)a.dgh + (long)t * 3 * NH + (long)n * 3 * H + g * H + c : (const T *)a.h + (long)t * NH + (long)n * H + c;
                constexpr int W = sizeof(T) / 2;
                u64 v[W] = {};
                for (int i = 0; i < wait / 4; ++i) __builtin_amdgcn_s_sleep(1);
                bool missing = true;
                for (bool first = true; missing && left > 0; first = false) {
                    bool un = false;
#pragma unroll
                    for (int e = 0; e < W; ++e) v[e] = seen((const char *)src + 8 * e);
#pragma unroll
                    for (int e = 0; e < W; ++e) un |= unset<T>(v[e]);
                    missing = __any(un);
                    if (missing) {
                        --left;
                        if (first && !near) wait = min(wait + kSleepUp, kSleepMost);
                    }
                }
                if (wait > 0) wait -= 1;
                gave_up |= missing;
#pragma unroll
                for (int e = 0; e < W; ++e) *(u64 *)((char *)(vec + (step & 1) * NV * HP + g * HP + c) + 8 * e) = v[e];
            }
            lds_barrier();
        }
        __syncthreads();           // (the block's units of the last row are stored)
        if (gave_up && c == 0) {
            T *last = BWD ? (T *)a.dgh + (long)n * 3 * H + u0 : (T *)a.h + (long)a.T * NH + (long)n * H + u0;
            *(typename ST::U *)last = (typename ST::U)kUnset;
        }
        return;
    }

    // part p = (unit slot + SLOTS*(p/3), gate p%3): byte offset of its row of this thread's columns; columns past H read zeros
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a.w, 0, (unsigned)(3 * H * H * (int)sizeof(T)), 0x00020000);
    auto row = [&](int p) -> unsigned {
        const int u = min(u0 + slot + SLOTS * (p / 3), H - 1), g = p % 3;
        return (unsigned)((BWD ? u * 3 * H + g * H : (g * H + u) * H) + 4 * q) * (unsigned)sizeof(T);
    };
    auto column = [&](int m) { return 4 * (q + 8 * m); };
    auto load = [&](unsigned r, int m) -> V {
        const unsigned at = r + (unsigned)(32 * m * (int)sizeof(T));
        if (32 * m + 32 <= 32 * (M - 2)) return ST::fetch(w_rsrc, at);     // (H > 32*(M - 2))
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
        for (int m = 0; m < M; ++m) lw[(p * M + m) * MT + tid] = load(row(RS + p), m);
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
    // (SPLIT: the second half is the pollers', who fill its first H columns at the second step; all read those past H)
    for (int i = tid; i < 2 * NV * HP; i += MT)
        if (!SPLIT || i < NV * HP || i % HP >= H) vec[i] = !BWD && SPLIT && i < H ? ((const T *)a.h)[(long)n * H + i] : (T)0.f;
    if constexpr (!SPLIT) __syncthreads();

    // this lane's unit in the elementwise part
    const int u = u0 + slot + SLOTS * q;
    const bool mine = q < IU && u < u1;
    const int ue = mine ? u : 0;
    const long at = (long)n * H + ue;
    float br = 0.f, bz = 0.f, bin = 0.f, bhn = 0.f, state = 0.f;   // state: h (forward), the direct part of dh (backward)
    if constexpr (!BWD) {
        br = a.b_ih[ue] + a.b_hh[ue];
        bz = a.b_ih[H + ue] + a.b_hh[H + ue];
        bin = a.b_ih[2 * H + ue];
        bhn = a.b_hh[2 * H + ue];
        state = (float)((const T *)a.h)[at];
        if constexpr (!SPLIT) {
            if (mine) vec[u] = (T)state;
            __syncthreads();
        }
    } else {
        state = (float)((const T *)a.dh_top)[at];
    }

    // The elementwise operands of a step, requested two steps ahead (they come from HBM, which takes longer than a step): 618 / 621 ->
    // 566 / 594 us at H = 256 without a split, 119 / 113 -> 95 / 88 at H = 40; only one ahead at 192 units in fp32, which
    // has no registers left for more (274 / 274, 288 / 288 with two).
    constexpr int NE = BWD ? 5 : 3, D = sizeof(T) == 4 && M == 6 ? 1 : 2;
    // Forward in fp32, four blocks: and the place that the step's value will go to, which brings its line into the XCD's L2 (50 samples of 256
    // units 286 -> 273 us; backward 301 -> 332, bf16 224 -> 240 and two blocks 457 -> 473, which need the registers or the loads' time).
    constexpr int NP = SPLIT && !BWD && sizeof(T) == 4 && IU == 1 ? 1 : 0;
    T e[D][NE + NP];
    auto operands = [&](T *to, int step) {
        const int t = BWD ? a.T - 1 - step : step;
        const T *p = BWD ? (const T *)a.saved_in + (long)t * 4 * NH + (long)n * 4 * H + ue : (const T *)a.gi + (long)t * 3 * NH + (long)n * 3 * H + ue;
#pragma unroll
        for (int i = 0; i < (BWD ? 4 : 3); ++i) to[i] = p[i * H];
        if constexpr (BWD) to[NE - 1] = ((const T *)a.h)[(long)t * NH + at];
        if constexpr (NP > 0) to[NE] = ((const T *)a.h)[(long)(t + 1) * NH + at];
    };
#pragma unroll
    for (int k = 0; k < D; ++k) operands(e[k], min(k, a.T - 1));

    for (int first = 0; first < a.T; first += D)
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const int step = first + k, t = BWD ? a.T - 1 - step : step, buf = step & 1;
        if (k > 0 && step >= a.T) break;
        T ec[NE];
        auto take = [&] {
#pragma unroll
            for (int i = 0; i < NE; ++i) ec[i] = e[k][i];
            if constexpr (NP > 0) asm volatile("" ::"v"(e[k][NE]));
        };
        if constexpr (D == 1 || SPLIT) take();     // (waits here for what was requested; without a split the products come first)
        if constexpr (D == 1) operands(e[k], min(step + 1, a.T - 1));
        if constexpr (SPLIT) lds_barrier();
        const bool near = SPLIT && *near_lds;
        float acc[S];
#pragma unroll
        for (int p = 0; p < S; ++p) acc[p] = 0.f;
        // (no step comes after the last one, whose products are skipped; in fp32 that branch would spill, and they are dropped)
        if (!BWD || sizeof(T) == 4 || step > 0) {
            const T *v0 = vec + buf * NV * HP;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                V v[NV];
#pragma unroll
                for (int g = 0; g < NV; ++g) v[g] = *(const V *)(v0 + g * HP + column(m));
#pragma unroll
                for (int p = 0; p < SS; ++p) {
                    acc[RS + LS + p] = ST::template mac<FOUR>(acc[RS + LS + p], sw[p], v[BWD ? (RS + LS + p) % 3 : 0]);
                    sw[p] = load(rs[p], (m + 1) % M);
                }
#pragma unroll
                for (int p = 0; p < RS; ++p) acc[p] = ST::template mac<FOUR>(acc[p], wr[p][m], v[BWD ? p % 3 : 0]);
#pragma unroll
                for (int p = 0; p < LS; ++p) acc[RS + p] = ST::template mac<FOUR>(acc[RS + p], lw[(p * M + m) * MT + tid], v[BWD ? (RS + p) % 3 : 0]);
                if constexpr (SS > 0) __builtin_amdgcn_sched_barrier(0);     // (or every piece of the step is fetched ahead, into scratch)
            }
        }
        if constexpr (BWD) {
#pragma unroll
            for (int i = 0; i < IU; ++i) {
                acc[i] = (acc[3 * i] + acc[3 * i + 1]) + acc[3 * i + 2];
                if (sizeof(T) == 4) acc[i] = step > 0 ? acc[i] : 0.f;
            }
        }
        constexpr int R = BWD ? IU : S;
#pragma unroll
        for (int p = 0; p < R; ++p) acc[p] = sum8(acc[p]);
        if constexpr (!(D == 1 || SPLIT)) take();
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
                const float r = gate_sigmoid((float)ec[0] + gr + br);
                const float z = gate_sigmoid((float)ec[1] + gz + bz);
                const float qq = gn + bhn;
                const float c = gate_tanh((float)ec[2] + bin + r * qq);
                const T hn = (T)((1.f - z) * c + z * state);
                state = (float)hn;
                T *const hp = (T *)a.h + (long)(t + 1) * NH + at;
                if constexpr (SPLIT) {
                    publish(hp, hn, near);
                } else {
                    vn[u] = hn;
                    *hp = hn;
                }
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
                const float r = (float)ec[0], z = (float)ec[1], c = (float)ec[2], qq = (float)ec[3];
                const float da_n = dh * (1.f - z) * (1.f - c * c);
                const float da_z = dh * ((float)ec[4] - c) * z * (1.f - z);
                const float da_r = da_n * qq * r * (1.f - r);
                state = (float)(T)(dh * z);
                const T tr = (T)da_r, tz = (T)da_z, tn = (T)(da_n * r);
                const long g0 = (long)t * 3 * NH + (long)n * 3 * H + u;
                T *dgi = (T *)a.dgi + g0, *dgh = (T *)a.dgh + g0;
                if constexpr (SPLIT) {
                    publish(dgh, tr, near);
                    publish(dgh + H, tz, near);
                    publish(dgh + 2 * H, tn, near);
                } else {
                    vn[u] = tr;
                    vn[HP + u] = tz;
                    vn[2 * HP + u] = tn;
                    dgh[0] = tr;
                    dgh[H] = tz;
                    dgh[2 * H] = tn;
                }
                dgi[0] = tr;
                dgi[H] = tz;
                dgi[2 * H] = (T)da_n;
            }
        }
        if constexpr (D > 1) operands(e[k], min(step + D, a.T - 1));
        if constexpr (!SPLIT) lds_barrier();
    }
    if constexpr (SPLIT) {         // a poller that gave up writes over what is stored here
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
}

__global__ void unset_kernel(u64 *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = ~0ull;
}

template <typename T, bool BWD, int IU, int M, int RS, int LS, int SLOTS, bool SPLIT> int launch(const GruSeqArgs &a, hipStream_t stream)
{
    constexpr int MT = 8 * SLOTS;
    const size_t smem = 2 * (BWD ? 3 : 1) * 32 * M * sizeof(T) + (size_t)LS * M * MT * 4 * sizeof(T) + (SPLIT ? 16 : 0);
    static std::atomic<unsigned long long> done{0};
    if (smem > 64 * 1024) {
        const int rc = allow_lds((const void *)gru_seq_kernel<T, BWD, IU, M, RS, LS, SLOTS, SPLIT>, smem, done);
        if (rc != NSK_OK) return rc;
    }
    if (SPLIT) {
        // rows that are exchanged: h[1..T), or all of dgh (H * sizeof(T) is a multiple of 8)
        const size_t row = (size_t)a.N * a.H * sizeof(T);
        u64 *p = (u64 *)(BWD ? (char *)a.dgh : (char *)a.h + row);
        const size_t words = (BWD ? 3 * (size_t)a.T : (size_t)a.T) * row / 8;
        hipLaunchKernelGGL(unset_kernel, dim3((unsigned)std::min<size_t>((words + 1023) / 1024, 2048)), dim3(256), 0, stream, p, words);
        const int rc = check_launch();
        if (rc != NSK_OK) return rc;
    }
    const int blocks = SPLIT ? ceil_div(a.N, 8) * 8 * a.G : a.N, threads = MT + (SPLIT ? 64 * (BWD ? 3 : 1) : 0);
    hipLaunchKernelGGL((gru_seq_kernel<T, BWD, IU, M, RS, LS, SLOTS, SPLIT>), dim3(blocks), dim3(threads), smem, stream, a);
    return check_launch();
}

// Whether a stream may use all `cus` compute units (a mask may take some away)
bool whole_chip(hipStream_t stream, int cus)
{
    uint32_t mask[32] = {0};
    if (hipExtStreamGetCUMask(stream, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    int n = 0;
    for (uint32_t m : mask) n += __builtin_popcount(m);
    return n >= cus;
}

// Blocks per sample.  The groups of an XCD must fit on its CUs side by side: 4 up to 64 samples, 2 up to 128.  Splitting pays where
// one CU cannot hold the weight, above 192 units: us for T = 200, forward / backward, without -> with: fp32, 50 samples of 256
// units 574 / 594 -> 277 / 314 (G = 4; all exchanges through memory 297 / 337, and so with G = 8, 32 samples: 313 / 293 but unsteady), 100
// samples 574 / 598 -> 460 / 455 (G = 2);
// bf16, 50 samples 330 / 290 -> 238 / 263, but G = 2 293 / 334; 192 units: fp32 274 / 274 -> 252 / 292, bf16 215 / 205 -> 217 / 263.
// The launches before and behind are paid back from the first steps on with G = 4, with G = 2 from 16 on (100 samples, 2, 8, 16 steps, without /
// with: 11.7 / 14.1, 28.8 / 30.3, 51.7 / 50.0; a single step has no launch behind).
int split_of(int dtype, int T, int N, int H, hipStream_t stream)
{
    if (H % 8 != 0 || H <= 192) return 1;    // (polled in whole 8-byte words)
    static std::atomic<int> cus[64];         // of each device, once known
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1;
    int c = cus[dev].load(std::memory_order_relaxed);
    if (c == 0) {
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 1;
        cus[dev].store(c, std::memory_order_relaxed);
    }
    const int forced = hooks().gru_split;
    int g = 4;
    while (g > 1 && (ceil_div(N, 8) * g > c / 8 || (forced > 0 && g > forced))) g /= 2;
    if (g == 2 && (dtype == NSK_BF16 || (T > 1 && T < 16))) g = 1;
    return g > 1 && whole_chip(stream, c) ? g : 1;
}

// Parts in registers and in LDS: what the register file takes without spilling (512 threads: 256 registers each, with the polling
// wavefronts 168).  fp32 at H > 192 and G = 1, forward / backward in us: 5 parts in registers 705 / 619, 4 parts 775 / 691, 3 parts
// 893 / 784; 6 spill: 807 / 862.  Thirty-two slots of twice the units (four wavefronts, one per SIMD, so that the gates' code
// is issued once per SIMD) are faster where they need no more than half of the registers: bf16, 50 samples, 64 / 128 units
// 143 / 111 and 158 / 169 -> 104 / 96 and 143 / 143, split at 256 units 248 / 298 -> 228 / 276; fp32, 64 units 114 / 105 -> 106 / 105,
// but 128 units 173 / 192 -> 199 / 196.
template <typename T, bool BWD, int M> int dispatch(GruSeqArgs &a, hipStream_t stream)
{
    constexpr bool F = sizeof(T) == 4;
    a.HU = ceil_div(a.H, a.G);
    if constexpr (M == 8) {
        if (a.G > 1) {
            int rc;
            if constexpr (F)
                rc = a.G == 4 ? launch<T, BWD, 1, M, 3, 0, 64, true>(a, stream) : launch<T, BWD, 2, M, 4, 2, 64, true>(a, stream);
            else
                rc = launch<T, BWD, 2, M, 6, 0, 32, true>(a, stream);
            if (rc != NSK_OK || a.T == 1) return rc;       // (one step exchanges nothing)
            a.G = 1;
            a.HU = a.H;
            a.unfinished = true;
        }
        return launch<T, BWD, 4, M, F ? 5 : 9, F ? 2 : 3, 64, false>(a, stream);
    } else if constexpr (M == 6) {
        return launch<T, BWD, 3, M, F ? 7 : 9, F ? 2 : 0, 64, false>(a, stream);
    } else if constexpr (M == 4 && F) {
        return launch<T, BWD, 2, M, 6, 0, 64, false>(a, stream);
    } else {
        return launch<T, BWD, M, M, 3 * M, 0, 32, false>(a, stream);
    }
}
template <bool BWD> int dispatch(int dtype, GruSeqArgs &a, hipStream_t stream)
{
    const int m = (a.H + 63) / 64;
    if (dtype == NSK_BF16) {
        switch (m) {
        case 1: return dispatch<bf16_t, BWD, 2>(a, stream);
        case 2: return dispatch<bf16_t, BWD, 4>(a, stream);
        case 3: return dispatch<bf16_t, BWD, 6>(a, stream);
        default: return dispatch<bf16_t, BWD, 8>(a, stream);
        }
    }
    switch (m) {
    case 1: return dispatch<float, BWD, 2>(a, stream);
    case 2: return dispatch<float, BWD, 4>(a, stream);
    case 3: return dispatch<float, BWD, 6>(a, stream);
    default: return dispatch<float, BWD, 8>(a, stream);
    }
}

// Above 256 units a block would read nearly all of the weight again in every step, which the step launches spread over the chip; N
// is at most the 256 that the step calls take, so one wave of blocks.
bool seq_kernel_takes(int H) { return H <= 256; }

}  // namespace
}  // namespace nsk

using namespace nsk;

extern "C" {

int nsk_gru_seq_blocks(int dtype, int T, int N, int H, void *stream)
{
    if (T <= 0 || N <= 0 || H <= 0 || (dtype != NSK_F32 && dtype != NSK_BF16) || !nsk_gru_step_supported(N, H) || !seq_kernel_takes(H)) return 0;
    return split_of(dtype, T, N, H, (hipStream_t)stream);
}

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
        a.G = split_of(dtype, T, N, H, (hipStream_t)stream);
        a.polls = hooks().gru_polls >= 0 ? hooks().gru_polls : kPolls;
        a.apart = hooks().gru_far ? 1 : 8;
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
        a.G = split_of(dtype, T, N, H, (hipStream_t)stream);
        a.polls = hooks().gru_polls >= 0 ? hooks().gru_polls : kPolls;
        a.apart = hooks().gru_far ? 1 : 8;
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
