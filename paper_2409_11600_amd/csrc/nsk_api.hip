// The C ABI of libnsk: host-side validation, workspace planning and dispatch to the kernels.
// Every check that can be made without touching the device is made before the first HIP call, so
// the error paths behave identically on a machine without a GPU.
#include <limits.h>
#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "nsk_internal.h"

namespace nsk {

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(hipError_t e) { g_last_hip_error = (int)e; }

namespace {

int out_extent(int in, int pad, int dil, int filt, int stride)
{
    const long span = (long)in + 2L * pad - (long)dil * (filt - 1) - 1;
    return span < 0 ? 0 : (int)(span / stride + 1);
}

// NSK_OK, NSK_ERR_NULL, NSK_ERR_BAD_DESC or NSK_ERR_UNSUPPORTED.  `need_output`: an empty output
// (P or Q = 0) is a bad descriptor for the compute calls, but legal for the extent query.
int conv_geometry(const nsk_conv_desc_t *d, ConvGeo *g, bool need_output)
{
    if (!d) return NSK_ERR_NULL;
    if (d->N < 1 || d->C < 1 || d->H < 1 || d->W < 1 || d->K < 1 || d->R < 1 || d->S < 1) return NSK_ERR_BAD_DESC;
    if (d->stride_h < 1 || d->stride_w < 1 || d->dil_h < 1 || d->dil_w < 1) return NSK_ERR_BAD_DESC;
    if (d->pad_h < 0 || d->pad_w < 0) return NSK_ERR_BAD_DESC;
    if (d->dtype != NSK_F32 && d->dtype != NSK_BF16) return NSK_ERR_BAD_DESC;
    if (d->layout != NSK_NCHW && d->layout != NSK_NHWC) return NSK_ERR_BAD_DESC;
    g->N = d->N; g->C = d->C; g->H = d->H; g->W = d->W; g->K = d->K; g->R = d->R; g->S = d->S;
    g->sh = d->stride_h; g->sw = d->stride_w; g->ph = d->pad_h; g->pw = d->pad_w; g->dh = d->dil_h; g->dw = d->dil_w;
    g->dtype = d->dtype; g->layout = d->layout; g->es = elem_size(d->dtype);
    g->P = out_extent(d->H, d->pad_h, d->dil_h, d->R, d->stride_h);
    g->Q = out_extent(d->W, d->pad_w, d->dil_w, d->S, d->stride_w);
    if (!need_output) return NSK_OK;
    if (g->P < 1 || g->Q < 1) return NSK_ERR_BAD_DESC;
    // Limits of this build: pixel counts index with 32-bit ints, tap tables hold 64 entries with
    // 16-bit offsets, NCHW conversion puts the batch on gridDim.z.
    const long long pix_in = (long long)d->N * d->H * d->W, pix_out = (long long)d->N * g->P * g->Q;
    if (pix_in >= INT_MAX || pix_out >= INT_MAX) return NSK_ERR_UNSUPPORTED;
    if ((long long)d->R * d->S > kMaxTaps) return NSK_ERR_UNSUPPORTED;
    // activations are addressed with 32-bit byte offsets through buffer descriptors
    if (pix_in * d->C * 4 >= 0xFFFFFFFFLL || pix_out * d->K * 4 >= 0xFFFFFFFFLL) return NSK_ERR_UNSUPPORTED;
    if ((long long)(d->R - 1) * d->dil_h > 30000 || (long long)(d->S - 1) * d->dil_w > 30000) return NSK_ERR_UNSUPPORTED;
    if ((long long)d->K * d->R * d->S * d->C >= INT_MAX) return NSK_ERR_UNSUPPORTED;
    if (d->layout == NSK_NCHW && d->N > 65535) return NSK_ERR_UNSUPPORTED;
    g->x_elems = (size_t)pix_in * d->C;
    g->y_elems = (size_t)pix_out * d->K;
    g->w_elems = (size_t)d->K * d->R * d->S * d->C;
    return NSK_OK;
}

// Geometry part of the backward-weight arguments (pointers and split sizes are set by the caller).
void wgrad_geometry(const ConvGeo &g, WgradArgs *a)
{
    a->Nimg = g.N; a->H = g.H; a->W = g.W; a->C = g.C; a->P = g.P; a->Q = g.Q; a->K = g.K;
    a->sh = g.sh; a->sw = g.sw; a->ph = g.ph; a->pw = g.pw;
    a->ntaps = g.R * g.S;
    a->L = g.N * g.P * g.Q;
    for (int r = 0; r < g.R; ++r)
        for (int s = 0; s < g.S; ++s) {
            a->off_h[r * g.S + s] = (short)(r * g.dh);
            a->off_w[r * g.S + s] = (short)(s * g.dw);
        }
}

// The bf16 3x3 64->64 kernel writes 147 KB of partial sums per block, which only a long reduction pays for.  Measured against
// the pipelined kernel (us): 100 k rows 23.3 / 21.4, 200 k 30.0 / 32.7, 400 k 44 / 56.
bool use_wgrad_halo(const ConvGeo &g, const WgradArgs &a)
{
    if (!wgrad_halo64_applicable(g.dtype, a) || hooks().no_halo) return false;
    return a.L >= (hooks().wh_min_rows >= 0 ? hooks().wh_min_rows : 150000);
}

// The fp32 64 -> 64 kernel that applies the activation on load gives every CU whole tiles of 8 image rows, 41 us each; ragged rounds of
// them are slower than a pass for the activation and the pipelined kernel behind it (us with statistics, 32x32, pass and pipelined / on load: N=16
// 22 / 42, 48 42.0 / 42.8, 64 49.3 / 46.5, 96 71 / 85, 128 88 / 87, 192 122 / 127, 256 157 / 167), and from three rounds on all are.  lean: for a call
// without room for the activation, whole rounds of any number.
bool takes_halo64_f32_act(const ConvGeo &g, const IgemmArgs &a, bool lean)
{
    if (hooks().igemm_tile != 0 || !halo64_f32_act_applicable(g.dtype, a)) return false;
    const long tiles = (long)a.Nimg * (a.Hs / 8);
    return hooks().halo64_always || ((lean || tiles <= 512) && (tiles + 255) / 256 * 256 * 100 <= tiles * 105);
}

// Its backward-weight sibling writes 147 KB of partial sums a block, up to 256 (us, as above: N=2 11 / 17, 16 24 / 31, 32 40 / 37, 64 57 / 54,
// 128 96 / 90, 256 178 / 163).  lean: also below.
bool takes_rows32_f32_act(const ConvGeo &g, const WgradArgs &a, bool lean)
{
    return !hooks().no_halo && rows32_f32_act_applicable(g.dtype, a) && (lean || a.L >= 32768 || hooks().halo64_always);
}

bool whole_vectors(const ConvGeo &g, int channels) { return channels % (g.dtype == NSK_BF16 ? 8 : 4) == 0; }

// The layer as the kernels see it: where the channels that the pass reads are not whole 16-byte vectors (of x in the forward
// pass, of dy backward, of both for the weights), the operands are copied into the workspace with zero channels up to the
// next whole one, and the kernels for whole vectors run: the copy is a pass at memory speed and a launch, where the
// element-wise kernels take 3 to 40 times their time.  Measured (us, element-wise / copy and whole vectors; forward, weights,
// backward): bf16 3x3 100->100 at 28x28 N=32 174, 125, 186 / 20, 29, 21; 300->300 stride 2 at 14x14 N=16 506, 45, 555 /
// 24, 22, 20; 1x1 20->100 at 28x28 N=64 28, 28, 36 / 14, 20, 15; 3x3 20->20 at 7x7 N=1 27, 11, 30 / 9, 9, 9; fp32 3x3 30->30 at
// 28x28 N=64 49, 49, 51 / 25, 38, 25.  Up to four channels have kernels of their own; 5 and 6 in fp32 gain nothing
// (3x3 5->48 at 56x56 N=64 36, 46, 76 / 51, 44, 75).
ConvGeo padded_geometry(const ConvGeo &g, int pass, int groups)
{
    const int vec = g.dtype == NSK_BF16 ? 8 : 4;
    const int least = g.dtype == NSK_BF16 ? 4 : 6;
    const bool pad_c = pass != NSK_PASS_DGRAD && !whole_vectors(g, g.C), pad_k = pass != NSK_PASS_FWD && !whole_vectors(g, g.K);
    if (groups > 1 || !(pad_c || pad_k) || stem_applicable(g) || hooks().no_pad) return g;
    if ((pad_c && g.C <= least) || (pad_k && g.K <= least)) return g;
    ConvGeo p = g;
    if (pad_c) p.C = ceil_div(g.C, vec) * vec;
    if (pad_k) p.K = ceil_div(g.K, vec) * vec;
    const size_t pix_in = (size_t)g.N * g.H * g.W, pix_out = (size_t)g.N * g.P * g.Q;
    p.x_elems = pix_in * p.C;
    p.y_elems = pix_out * p.K;
    p.w_elems = (size_t)p.K * g.R * g.S * p.C;
    // (the limits of conv_geometry)
    if (p.x_elems * 4 >= 0xFFFFFFFFull || p.y_elems * 4 >= 0xFFFFFFFFull || p.w_elems >= (size_t)INT_MAX) return g;
    return p;
}

// Workspace segments (byte offsets, each 256-aligned).
struct ConvPlan {
    ConvGeo geo;         // the layer as the kernels see it
    size_t act_in = 0;   // NHWC copy of the NCHW input activation (x or dy), or its copy with whole channel vectors
    size_t act_in2 = 0;  // wgrad only: the same of dy
    size_t filt = 0;     // packed filter
    size_t act_out = 0;  // NHWC result before conversion to NCHW
    size_t part = 0;     // wgrad partial sums
    size_t total = 0;
    int splits = 1, rows_per_split = 0;
    bool halo = false;   // wgrad: the 3x3 64->64 kernel writes one partial per block
    bool pipe = false;   // wgrad: the pipelined kernel
    bool grouped8 = false;   // wgrad: the kernel for groups of eight channels
    bool narrow = false;     // wgrad: the 3x3 kernel for 16 channels
    bool stem = false;   // the space-to-depth path plans its own workspace
    size_t act_tmp = 0;  // calls that take a raw input, on a kernel without a load that applies the activation: the applied activation
    bool act_fused = false;
};

// groups > 1: grouped convolution (the filter holds C/groups input channels per output channel and only the generic
// kernels run it).
void fwd_geometry(const ConvGeo &g, IgemmArgs *a);

// act: the call applies a batch-norm + ReLU to x (NHWC, one group): on load where a kernel for the layer does that, else into the workspace.
// lean: with as little workspace as the kernels for such a call can do with.
ConvPlan plan_conv(const ConvGeo &desc, int pass, int groups = 1, bool act = false, bool pad = true, bool lean = false)
{
    ConvPlan p;
    const ConvGeo g = pad ? padded_geometry(desc, pass, groups) : desc;
    p.geo = g;
    const bool pad_c = g.C != desc.C, pad_k = g.K != desc.K;
    const size_t w_elems = g.w_elems / (size_t)groups;
    p.stem = groups == 1 && stem_applicable(g);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes);
        return at;
    };
    if (act) {
        // (the pointers only matter for alignment tests: every tensor of these calls is 16-byte aligned)
        if (pass == NSK_PASS_FWD && !p.stem) {
            IgemmArgs a{};
            fwd_geometry(g, &a);
            p.act_fused = takes_halo64_f32_act(g, a, lean);
        } else if (pass == NSK_PASS_WGRAD && !p.stem) {
            WgradArgs wa{};
            wgrad_geometry(g, &wa);
            p.act_fused = takes_rows32_f32_act(g, wa, lean);
        }
        if (!p.act_fused) p.act_tmp = take(desc.x_elems * g.es);
    }
    if (p.stem) {
        p.total = off + stem_workspace_bytes(g, pass);
        return p;
    }
    const bool nchw = g.layout == NSK_NCHW;
    if (pass == NSK_PASS_FWD) {
        if (nchw || pad_c) {
            p.act_in = take(g.x_elems * g.es);
            p.filt = take(w_elems * g.es);
        }
        if (nchw) p.act_out = take(g.y_elems * g.es);
    } else if (pass == NSK_PASS_DGRAD) {
        if (nchw || pad_k) p.act_in = take(g.y_elems * g.es);
        // one packed filter per stride parity class; together they hold every tap once
        p.filt = take(w_elems * g.es + 256 * (size_t)g.sh * g.sw);
        if (nchw) p.act_out = take(g.x_elems * g.es);
    } else {
        if (nchw || pad_c) p.act_in = take(g.x_elems * g.es);
        if (nchw || pad_k) p.act_in2 = take(g.y_elems * g.es);
        WgradArgs wa{};
        wgrad_geometry(g, &wa);
        p.halo = groups == 1 && !p.act_fused && use_wgrad_halo(g, wa);
        if (p.act_fused)
            p.splits = rows32_f32_act_partials(wa, nullptr);
        else if (p.halo)
            p.splits = wgrad_halo64_partials(wa, nullptr);
        else {
            WgradArgs one = wa;   // one group's problem (aligned pointers and a split count stand for every launch)
            one.C = g.C / groups; one.K = g.K / groups;
            one.groups = groups; one.ldx = g.C; one.ldy = g.K;
            one.splits = 1;
            p.grouped8 = grouped8_wgrad_applicable(g.dtype, one);
            p.narrow = narrow_wgrad_applicable(g.dtype, one);
            const bool direct = p.grouped8 || p.narrow || tiny_wgrad_applicable(g.dtype, one) || (!hooks().no_depthwise && depthwise_wgrad_applicable(g.dtype, one));
            p.pipe = !direct && wgrad_pipe_applicable(g.dtype, one.C, one.K, groups);
            if (p.grouped8)
                p.splits = grouped8_wgrad_splits(one);
            else if (p.narrow)
                p.splits = narrow_wgrad_splits(one);
            else if (p.pipe)
                p.rows_per_split = wgrad_pipe_rows_per_split(g.dtype, one.L, one.K, one.ntaps * one.C, groups, &p.splits);
            else
                p.rows_per_split = wgrad_rows_per_split(g.dtype, one.L, g.K, one.ntaps * one.C, &p.splits);
        }
        if (!p.pipe && !p.grouped8 && groups > 1 && g.C == g.K && (g.C == groups || g.C == 2 * groups || g.C == 4 * groups || g.C == 8 * groups)) {
            // depthwise and its neighbours: the direct kernel runs blocks of 16 channel vectors x one split and wants
            // about four per CU
            const int vec = g.dtype == NSK_BF16 ? 8 : 4, L = g.N * g.P * g.Q;
            const int want = 1024 / ceil_div(ceil_div(g.C, vec), 16) > 0 ? 1024 / ceil_div(ceil_div(g.C, vec), 16) : 1;
            int rows = ceil_div(L, want);
            if (rows < 64) rows = 64;
            p.rows_per_split = ceil_div(rows, 32) * 32;
            p.splits = ceil_div(L, p.rows_per_split);
        }
        // a grouped launch puts groups * splits on gridDim.z
        while (!p.pipe && !p.grouped8 && (long)groups * p.splits > 65535) {
            p.rows_per_split *= 2;
            p.splits = ceil_div(g.N * g.P * g.Q, p.rows_per_split);
        }
        p.part = take((size_t)p.splits * w_elems * sizeof(float));
    }
    p.total = off;
    return p;
}

// The plan of a call: where the workspace is too small for the copies with whole channel vectors (an NHWC forward pass on the
// operands as they lie needs none at all), the element-wise kernels take the layer; where it is too small for an applied activation, the kernel that
// applies it on load, if there is one.
ConvPlan plan_within(const ConvGeo &desc, int pass, int groups, bool act, const void *ws, size_t have)
{
    const ConvPlan p = plan_conv(desc, pass, groups, act);
    if ((ws ? have : 0) >= p.total || ((!act || p.act_fused) && p.geo.C == desc.C && p.geo.K == desc.K)) return p;
    const ConvPlan q = plan_conv(desc, pass, groups, act, false, true);
    return q.total <= (ws ? have : 0) ? q : p;
}

bool misaligned(const void *p) { return ((uintptr_t)p & 15) != 0; }

int check_ws(const void *ws, size_t have, size_t need)
{
    if (need == 0) return NSK_OK;
    if (!ws || have < need) return NSK_ERR_WORKSPACE;
    if (misaligned(ws)) return NSK_ERR_ALIGNMENT;
    return NSK_OK;
}

#define NSK_TRY(expr)                 \
    do {                              \
        const int st__ = (expr);      \
        if (st__ != NSK_OK) return st__; \
    } while (0)

int bn_geometry(const nsk_bn_desc_t *d)
{
    if (!d) return NSK_ERR_NULL;
    if (d->N < 1 || d->C < 1 || d->H < 1 || d->W < 1) return NSK_ERR_BAD_DESC;
    if (d->dtype != NSK_F32 && d->dtype != NSK_BF16) return NSK_ERR_BAD_DESC;
    if (d->layout != NSK_NCHW && d->layout != NSK_NHWC) return NSK_ERR_BAD_DESC;
    if (!(d->eps >= 0.f) || !(d->momentum >= 0.f && d->momentum <= 1.f)) return NSK_ERR_BAD_DESC;
    if (d->relu != 0 && d->relu != 1) return NSK_ERR_BAD_DESC;
    if (d->C > 65535) return NSK_ERR_UNSUPPORTED;
    return NSK_OK;
}

int pool_geometry(const nsk_pool_desc_t *d, int *P, int *Q)
{
    if (!d) return NSK_ERR_NULL;
    if (d->N < 1 || d->C < 1 || d->H < 1 || d->W < 1 || d->R < 1 || d->S < 1) return NSK_ERR_BAD_DESC;
    if (d->stride_h < 1 || d->stride_w < 1 || d->pad_h < 0 || d->pad_w < 0) return NSK_ERR_BAD_DESC;
    if (d->dtype != NSK_F32 && d->dtype != NSK_BF16) return NSK_ERR_BAD_DESC;
    if (d->layout != NSK_NCHW && d->layout != NSK_NHWC) return NSK_ERR_BAD_DESC;
    if ((long)d->R * d->S > 127) return NSK_ERR_UNSUPPORTED;
    *P = out_extent(d->H, d->pad_h, 1, d->R, d->stride_h);
    *Q = out_extent(d->W, d->pad_w, 1, d->S, d->stride_w);
    return NSK_OK;
}

// Geometry part of the forward implicit-GEMM arguments (pointers, byte sizes and statistics are set by the caller).
void fwd_geometry(const ConvGeo &g, IgemmArgs *a)
{
    a->Nimg = g.N; a->Hs = g.H; a->Ws = g.W; a->Cs = g.C;
    a->Mi = g.P; a->Mj = g.Q; a->M = g.N * g.P * g.Q;
    a->mult_h = g.sh; a->add_h = -g.ph; a->mult_w = g.sw; a->add_w = -g.pw;
    a->ntaps = g.R * g.S; a->Ktot = a->ntaps * g.C;
    a->Ngemm = g.K;
    a->Ho = g.P; a->Wo = g.Q; a->Co = g.K; a->osh = 1; a->oa = 0; a->osw = 1; a->ob = 0;
    a->accumulate = 0;
    a->src_bytes = (unsigned)(g.x_elems * g.es);
    a->wpk_bytes = (unsigned)(g.w_elems * g.es);
    for (int r = 0; r < g.R; ++r)
        for (int s = 0; s < g.S; ++s) {
            a->off_h[r * g.S + s] = (short)(r * g.dh);
            a->off_w[r * g.S + s] = (short)(s * g.dw);
        }
}

// The output tensor of a convolution as a batch-norm descriptor of its NHWC form (what the kernels write).
nsk_bn_desc_t output_as_bn(const ConvGeo &g)
{
    nsk_bn_desc_t d{};
    d.N = g.N; d.C = g.K; d.H = g.P; d.W = g.Q;
    d.dtype = g.dtype; d.layout = NSK_NHWC;
    d.eps = 0.f; d.momentum = 0.f; d.relu = 0;
    return d;
}

// Rows of partial sums nsk_conv2d_fwd_stats writes: those of the kernel's own epilogue where it has one (*fused),
// else those of the separate reduction pass over the stored output.
int conv_stats_rows(const ConvGeo &g, bool *fused = nullptr)
{
    int rows = 0;
    if (stem_applicable(g)) {
        rows = stem_stats_rows(g);
    } else {
        IgemmArgs a{};
        fwd_geometry(padded_geometry(g, NSK_PASS_FWD, 1), &a);
        rows = igemm_stats_rows(g.dtype, a);
    }
    if (fused) *fused = rows > 0;
    return rows > 0 ? rows : bn_stats_rows(output_as_bn(g));
}

// NSK_OK if C and K split into `groups` equal runs.
int check_groups(const ConvGeo &g, int groups)
{
    if (groups < 1 || g.C % groups != 0 || g.K % groups != 0) return NSK_ERR_BAD_DESC;
    if (groups > 65535) return NSK_ERR_UNSUPPORTED;   // groups ride on gridDim.z
    return NSK_OK;
}

// The input of a fused-activation call as a batch-norm descriptor.
nsk_bn_desc_t input_as_bn(const ConvGeo &g)
{
    nsk_bn_desc_t d{};
    d.N = g.N; d.C = g.C; d.H = g.H; d.W = g.W;
    d.dtype = g.dtype; d.layout = NSK_NHWC;
    d.eps = 0.f; d.momentum = 0.f; d.relu = 1;
    return d;
}

// NSK_OK if the fused-activation calls take this layer: NHWC, one group, channels the vector kernels handle.
int check_act(const ConvGeo &g, int groups, const float *act)
{
    if (!act) return NSK_OK;
    if (misaligned(act)) return NSK_ERR_ALIGNMENT;
    if (g.layout != NSK_NHWC || groups != 1 || !bn_act_supported(input_as_bn(g))) return NSK_ERR_UNSUPPORTED;
    return NSK_OK;
}

int conv_fwd_impl(const nsk_conv_desc_t *desc, int groups, const void *x, const void *w, void *y, float *stats,
                  void *workspace, size_t workspace_bytes, void *stream, const float *act = nullptr)
{
    ConvGeo g;
    NSK_TRY(conv_geometry(desc, &g, true));
    NSK_TRY(check_groups(g, groups));
    if (!x || !w || !y) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(w) || misaligned(y)) return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_act(g, groups, act));
    const ConvPlan p = plan_within(g, NSK_PASS_FWD, groups, act != nullptr, workspace, workspace_bytes);
    const int cg = g.C / groups, kg = g.K / groups;
    NSK_TRY(check_ws(workspace, workspace_bytes, p.total));
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    if (act && !p.act_fused) {   // the kernel for this layer does not apply the activation on load
        NSK_TRY(launch_bn_act(input_as_bn(g), x, act, ws + p.act_tmp, st));
        x = ws + p.act_tmp;
        if (p.stem) ws += align_up(g.x_elems * g.es);
    }
    bool fused = false;
    const int rows = stats ? conv_stats_rows(g, &fused) : 0;
    if (p.geo.C == g.C && padded_geometry(g, NSK_PASS_FWD, groups).C != g.C) fused = false;   // (rows: what the query answered)
    if (p.stem) {
        void *y_nhwc = nullptr;
        NSK_TRY(stem_fwd(g, x, w, y, ws, fused ? stats : nullptr, rows, &y_nhwc, st));
        if (stats && !fused) NSK_TRY(launch_bn_stats(output_as_bn(g), y_nhwc, stats, rows, st));
        return NSK_OK;
    }

    const void *src = x, *filt = w;
    void *dst = y;
    const ConvGeo &gp = p.geo;
    const bool nchw = g.layout == NSK_NCHW;
    if (nchw || gp.C != g.C) {
        if (nchw)
            NSK_TRY(launch_nchw_to_nhwc(g.dtype, x, ws + p.act_in, g.N, g.C, g.H, g.W, gp.C, st));
        else
            NSK_TRY(launch_pad_channels(g.dtype, x, ws + p.act_in, (long)g.N * g.H * g.W, g.C, gp.C, st));
        int tap_off[kMaxTaps];
        for (int t = 0; t < g.R * g.S; ++t) tap_off[t] = nchw ? t : t * cg;
        NSK_TRY(launch_pack_filter(g.dtype, w, ws + p.filt, g.K, g.R * g.S, gp.C / groups, cg, (long)cg * g.R * g.S,
                                   nchw ? (long)g.R * g.S : 1L, tap_off, st));
        src = ws + p.act_in;
        filt = ws + p.filt;
        if (nchw) dst = ws + p.act_out;
    }
    IgemmArgs a{};
    fwd_geometry(gp, &a);
    a.src = src; a.wpk = filt; a.out = dst;
    if (groups > 1) {   // `groups` problems of cg -> kg channels on channel runs of the same tensors
        a.groups = groups;
        a.src_ld = g.C;
        a.Cs = cg;
        a.Ktot = a.ntaps * cg;
        a.Ngemm = kg;
        a.wpk_bytes = (unsigned)(g.w_elems / (size_t)groups * g.es);
    }
    if (p.act_fused) {
        NSK_TRY(launch_halo64_f32_act(a, act, fused ? stats : nullptr, rows, st));
        return stats && !fused ? launch_bn_stats(output_as_bn(g), dst, stats, rows, st) : NSK_OK;
    }
    if (fused) {
        a.stats = stats;
        a.stats_rows = rows;
    }
    NSK_TRY(launch_igemm(g.dtype, a, st));
    if (stats && !fused) NSK_TRY(launch_bn_stats(output_as_bn(g), dst, stats, rows, st));
    if (nchw) NSK_TRY(launch_nhwc_to_nchw(g.dtype, dst, y, g.N, g.K, g.P, g.Q, 0, st));
    return NSK_OK;
}

}  // namespace
}  // namespace nsk

using namespace nsk;

namespace nsk {
namespace {
TestHooks g_hooks;
bool g_hooks_read = false;

void read_hooks()
{
    auto on = [](const char *name) { return getenv(name) != nullptr; };
    auto num = [](const char *name) { const char *e = getenv(name); return e ? atoll(e) : -1LL; };
    TestHooks h{};
    h.no_pw = on("NSK_NO_PW");
    h.no_halo = on("NSK_NO_HALO");
    h.gru_far = on("NSK_GRU_FAR");
    h.no_fs = on("NSK_NO_FS");
    h.no_halo_wide = on("NSK_NO_HALO_WIDE");
    h.halo_wide_always = on("NSK_HALO_WIDE_ALWAYS");
    h.halo64_always = on("NSK_HALO64_ALWAYS");
    h.halo_single = on("NSK_HALO_SINGLE");
    h.no_stem = on("NSK_NO_STEM");
    h.no_stem_halo = on("NSK_NO_STEM_HALO");
    h.no_tiny = on("NSK_NO_TINY");
    h.no_depthwise = on("NSK_NO_DEPTHWISE");
    h.no_grouped8 = on("NSK_NO_GROUPED8");
    h.no_pad = on("NSK_NO_PAD");
    h.depthwise_no_rows = on("NSK_DEPTHWISE_NO_ROWS");
    h.depthwise_no_cols = on("NSK_DEPTHWISE_NO_COLS");
    h.pool_general = on("NSK_POOL_GENERAL");
    h.reduce4 = on("NSK_REDUCE4");
    h.wh_no_split = on("NSK_WH_NO_SPLIT");
    h.pw_min_rows = num("NSK_PW_MIN_ROWS");
    h.wh_min_rows = num("NSK_WH_MIN_ROWS");
    const long long tile = num("NSK_IGEMM_TILE");
    h.igemm_tile = tile > 0 ? (int)tile : 0;
    const long long split = num("NSK_GRU_SPLIT");
    h.gru_split = split > 0 ? (int)split : 0;
    const long long polls = num("NSK_GRU_POLLS");
    h.gru_polls = polls >= 0 && polls <= INT_MAX ? (int)polls : -1;
    g_hooks = h;
    g_hooks_read = true;
}
}  // namespace

const TestHooks &hooks()
{
    if (!g_hooks_read) read_hooks();
    return g_hooks;
}
}  // namespace nsk

extern "C" {

int nsk_version(void) { return 100; }

void nsk_test_hooks_reload(void) { nsk::read_hooks(); }

const char *nsk_status_string(int status)
{
    switch (status) {
    case NSK_OK: return "ok";
    case NSK_ERR_NULL: return "a required pointer is NULL";
    case NSK_ERR_BAD_DESC: return "descriptor field out of range or empty output";
    case NSK_ERR_UNSUPPORTED: return "valid request not supported by this build";
    case NSK_ERR_WORKSPACE: return "workspace missing or too small";
    case NSK_ERR_ALIGNMENT: return "pointer not 16-byte aligned";
    case NSK_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
    }
}

int nsk_last_hip_error(void) { return g_last_hip_error; }

int nsk_conv2d_out_dims(const nsk_conv_desc_t *desc, int *P, int *Q)
{
    if (!desc || !P || !Q) return NSK_ERR_NULL;
    ConvGeo g;
    NSK_TRY(conv_geometry(desc, &g, false));
    *P = g.P;
    *Q = g.Q;
    return NSK_OK;
}

size_t nsk_conv2d_workspace_bytes(const nsk_conv_desc_t *desc, int pass)
{
    ConvGeo g;
    if (pass < NSK_PASS_FWD || pass > NSK_PASS_WGRAD) return 0;
    if (conv_geometry(desc, &g, true) != NSK_OK) return 0;
    return plan_conv(g, pass).total;
}

int nsk_conv2d_fwd(const nsk_conv_desc_t *desc, const void *x, const void *w, void *y, void *workspace,
                   size_t workspace_bytes, void *stream)
{
    return conv_fwd_impl(desc, 1, x, w, y, nullptr, workspace, workspace_bytes, stream);
}

int nsk_conv2d_stats_rows(const nsk_conv_desc_t *desc)
{
    ConvGeo g;
    if (conv_geometry(desc, &g, true) != NSK_OK) return 0;
    return conv_stats_rows(g);
}

int nsk_conv2d_fwd_stats(const nsk_conv_desc_t *desc, const void *x, const void *w, void *y, float *stats,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    if (!stats) return NSK_ERR_NULL;
    if (misaligned(stats)) return NSK_ERR_ALIGNMENT;
    return conv_fwd_impl(desc, 1, x, w, y, stats, workspace, workspace_bytes, stream);
}

// Layers whose filters are packed together (launch_pack_many) / whose partial sums are added up together: the calls below need no
// workspace for them.
static bool packs_with_others(const ConvGeo &g)
{
    const ConvPlan p = plan_conv(g, NSK_PASS_DGRAD);
    return g.layout == NSK_NHWC && !p.stem && p.geo.C == g.C && p.geo.K == g.K && g.R * g.S <= 9 && g.sh * g.sw <= 4 && g.w_elems < 140000;
}
static bool reduces_with_others(const ConvGeo &g, const ConvPlan &p)
{
    return g.layout == NSK_NHWC && !p.stem && p.geo.C == g.C && p.geo.K == g.K && p.splits > 1 &&
           (size_t)p.splits * g.w_elems * sizeof(float) <= (16u << 20);
}

// packed: the filter is there already (packs_with_others).  collect: nothing is launched, the packings of w into `packed` are appended.
static int conv_dgrad_impl(const nsk_conv_desc_t *desc, int groups, const void *dy, const void *w, void *dx,
                           int accumulate, void *workspace, size_t workspace_bytes, void *stream, void *packed = nullptr,
                           std::vector<PackItem> *collect = nullptr)
{
    ConvGeo g;
    NSK_TRY(conv_geometry(desc, &g, true));
    NSK_TRY(check_groups(g, groups));
    if (!dy || !w || !dx) return NSK_ERR_NULL;
    if (accumulate != 0 && accumulate != 1) return NSK_ERR_BAD_DESC;
    if (misaligned(dy) || misaligned(w) || misaligned(dx) || misaligned(packed)) return NSK_ERR_ALIGNMENT;
    if (packed && !packs_with_others(g)) return NSK_ERR_UNSUPPORTED;
    const ConvPlan p = plan_within(g, NSK_PASS_DGRAD, groups, false, workspace, workspace_bytes);
    const ConvGeo &gp = p.geo;
    const int cg = g.C / groups, kg = gp.K / groups;   // channels of one group (all of them for a plain convolution)
    if (!packed) NSK_TRY(check_ws(workspace, workspace_bytes, p.total));
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    char *const filters = packed ? (char *)packed : ws + p.filt;
    const bool nchw = g.layout == NSK_NCHW;
    if (p.stem) return stem_dgrad(g, dy, w, dx, accumulate, ws, st);

    const void *src = dy;
    void *dst = dx;
    int acc_kernel = accumulate;
    if (nchw) {
        NSK_TRY(launch_nchw_to_nhwc(g.dtype, dy, ws + p.act_in, g.N, g.K, g.P, g.Q, gp.K, st));
        src = ws + p.act_in;
        dst = ws + p.act_out;
        acc_kernel = 0;  // the conversion back to NCHW does the add
    } else if (gp.K != g.K) {
        NSK_TRY(launch_pad_channels(g.dtype, dy, ws + p.act_in, (long)g.N * g.P * g.Q, g.K, gp.K, st));
        src = ws + p.act_in;
    }
    // dx[h] with h = a + sh*i receives dy[p] * w[r] exactly for the taps r with
    // (a + ph - r*dh) divisible by sh, at p = i + (a + ph - r*dh)/sh: one dense sub-problem per
    // residue class (a, b) of (h mod sh, w mod sw), so no multiply is spent on inserted zeros.
    // Geometry of one class (everything but the pointers); returns its number of taps.
    auto class_args = [&](int ca, int cb, IgemmArgs *a, int *tap_off) {
        int nt = 0;
        for (int r = 0; r < g.R; ++r) {
            const int th = ca + g.ph - r * g.dh;
            if (((th % g.sh) + g.sh) % g.sh != 0) continue;
            for (int s = 0; s < g.S; ++s) {
                const int tw = cb + g.pw - s * g.dw;
                if (((tw % g.sw) + g.sw) % g.sw != 0) continue;
                a->off_h[nt] = (short)(th / g.sh);  // exact division, may be negative
                a->off_w[nt] = (short)(tw / g.sw);
                tap_off[nt] = nchw ? r * g.S + s : (r * g.S + s) * cg;
                ++nt;
            }
        }
        a->Nimg = g.N; a->Hs = g.P; a->Ws = g.Q; a->Cs = kg;
        a->Mi = ca < g.H ? (g.H - ca + g.sh - 1) / g.sh : 0;
        a->Mj = cb < g.W ? (g.W - cb + g.sw - 1) / g.sw : 0;
        a->M = g.N * a->Mi * a->Mj;
        a->mult_h = 1; a->add_h = 0; a->mult_w = 1; a->add_w = 0;
        a->ntaps = nt; a->Ktot = nt * kg;
        a->Ngemm = cg;
        if (groups > 1) {
            a->groups = groups;
            a->src_ld = g.K;   // (grouped layers are not padded)
        }
        a->Ho = g.H; a->Wo = g.W; a->Co = g.C; a->osh = g.sh; a->oa = ca; a->osw = g.sw; a->ob = cb;
        a->accumulate = acc_kernel;
        a->src_bytes = (unsigned)(gp.y_elems * g.es);
        a->wpk_bytes = (unsigned)((size_t)g.C * nt * kg * g.es);
        return nt;
    };
    // Stride 2 with every tap in class (0, 0) (a 1x1 layer): the other three classes are plain zeros, which the
    // short-reduction kernel writes along with class (0, 0) when it takes that class.
    bool zero_cell = false;
    if (g.sh == 2 && g.sw == 2 && !acc_kernel && groups == 1) {
        IgemmArgs a{};
        int tap_off[kMaxTaps];
        bool others_empty = true;
        for (int c = 1; c < 4; ++c) others_empty = others_empty && class_args(c >> 1, c & 1, &a, tap_off) == 0;
        if (others_empty && class_args(0, 0, &a, tap_off) > 0) {
            a.src = src; a.wpk = filters; a.out = dst;
            zero_cell = conv_pw_applicable(g.dtype, a);
        }
    }
    // element (k, tap, c) of the filter: k * w_sc + tap_off + c * w_sn; one group's filters are w_gstep elements long
    const long w_sn = nchw ? (long)g.R * g.S : 1L, w_sc = (long)g.R * g.S * cg;
    const int kr = g.K / groups;
    const long w_gstep = (long)kr * w_sc;
    size_t filt_off = 0;
    // classes with taps: filters are packed first, then the launches follow (one for all classes where the pipelined
    // kernel takes them together)
    IgemmArgs pending[4], zeros[4];
    int n_pending = 0, n_zeros = 0;
    const bool may_merge = g.sh * g.sw <= 4;
    int pk_taps[4][kMaxTaps], pk_nt[4];
    void *pk_out[4];
    for (int ca = 0; ca < g.sh; ++ca)
        for (int cb = 0; cb < g.sw; ++cb) {
            IgemmArgs a{};
            int tap_off[kMaxTaps];
            const int nt = class_args(ca, cb, &a, tap_off);
            if (a.Mi == 0 || a.Mj == 0) continue;
            if (nt == 0 && accumulate && !nchw) continue;  // nothing to add
            if (nt == 0) {   // no tap reaches this class: plain zero fill
                if (may_merge) {
                    a.src = src; a.wpk = filters; a.out = dst;
                    if (!zero_cell) zeros[n_zeros++] = a;
                } else {
                    NSK_TRY(launch_zero_class(g.dtype, dst, g.N, g.H, g.W, g.C, a.Mi, a.Mj, g.sh, ca, g.sw, cb, st));
                }
                continue;
            }
            // packed filter of this class: [c][tap][k] with element (c, t, k) = w[c*sn + tap_off[t] + k*sc]
            a.src = src; a.wpk = filters + filt_off; a.out = dst;
            a.zero_cell = zero_cell ? 1 : 0;
            a.packed = !packed;
            if (may_merge) {
                for (int t = 0; t < kMaxTaps; ++t) pk_taps[n_pending][t] = t < nt ? tap_off[t] : 0;
                pk_nt[n_pending] = nt;
                pk_out[n_pending] = filters + filt_off;
                pending[n_pending++] = a;
            } else {
                int taps1[1][kMaxTaps];
                for (int t = 0; t < kMaxTaps; ++t) taps1[0][t] = t < nt ? tap_off[t] : 0;
                void *out1[1] = {filters + filt_off};
                NSK_TRY(launch_pack_filters_grouped(g.dtype, 1, w, out1, cg, &nt, kg, kr, w_sn, w_sc, taps1, groups, w_gstep, st));
                NSK_TRY(launch_igemm(g.dtype, a, st));
            }
            filt_off += align_up((size_t)g.C * nt * kg * g.es);
        }
    if (collect) {
        for (int i = 0; i < n_pending; ++i) {
            PackItem e{w, pk_out[i], cg, pk_nt[i], kg, (int)w_sn, (int)w_sc, 0, {}};
            for (int t = 0; t < pk_nt[i]; ++t) e.tap_off[t] = pk_taps[i][t];
            collect->push_back(e);
        }
        return NSK_OK;
    }
    // Small fp32 layers whose launch is that of the pipelined kernel: it fetches the filter itself, and no packing goes before it.  (The classes
    // without a tap count for the tile as they do in the launch on a packed filter: the same sums in the same order.)
    const bool one_launch = n_pending + n_zeros <= 4 && n_pending > 0 && !nchw && groups == 1 && !packed;
    if (one_launch) std::copy(zeros, zeros + n_zeros, pending + n_pending);
    if (one_launch && igemm_pipe_multi_applicable(g.dtype, pending, n_pending) && igemm_pipe_gathers(g.dtype, pending, n_pending + n_zeros)) {
        for (int i = 0; i < n_pending; ++i) {
            pending[i].gather = 1;
            pending[i].wpk = w;
            pending[i].wpk_bytes = (unsigned)(g.w_elems * g.es);   // (channels added to whole vectors read zeros past the end)
            pending[i].w_sc = (int)w_sc;
            for (int t = 0; t < pk_nt[i]; ++t) pending[i].w_tap[t] = (unsigned char)(pk_taps[i][t] / cg);
        }
        for (int i = 0; i < n_zeros; ++i) pending[n_pending + i].gather = 1;
        return launch_igemm_pipe_multi(g.dtype, pending, n_pending + n_zeros, st);
    }
    // one packing launch for all classes, then their multiplies
    if (n_pending > 0 && !packed)
        NSK_TRY(launch_pack_filters_grouped(g.dtype, n_pending, w, pk_out, cg, pk_nt, kg, kr, w_sn, w_sc, pk_taps, groups, w_gstep, st));
    if (n_pending == 4 && groups == 1 && fs64_dgrad_s2_applicable(g.dtype, pending, n_pending)) {
        NSK_TRY(launch_fs64_dgrad_s2(pending, n_pending, st));
    } else if (n_pending > 1 && groups == 1 && halo_wide_multi_applicable(g.dtype, pending, n_pending)) {
        NSK_TRY(launch_halo_wide_multi(pending, n_pending, st));
    } else if (n_pending + n_zeros > 1 && n_pending > 0 && igemm_pipe_multi_applicable(g.dtype, pending, n_pending)) {
        for (int i = 0; i < n_zeros; ++i) pending[n_pending + i] = zeros[i];
        NSK_TRY(launch_igemm_pipe_multi(g.dtype, pending, n_pending + n_zeros, st));
        n_zeros = 0;
    } else {
        for (int i = 0; i < n_pending; ++i) NSK_TRY(launch_igemm(g.dtype, pending[i], st));
    }
    for (int i = 0; i < n_zeros; ++i)
        NSK_TRY(launch_zero_class(g.dtype, dst, g.N, g.H, g.W, g.C, zeros[i].Mi, zeros[i].Mj, g.sh, zeros[i].oa, g.sw, zeros[i].ob, st));
    if (nchw) NSK_TRY(launch_nhwc_to_nchw(g.dtype, dst, dx, g.N, g.C, g.H, g.W, accumulate, st));
    return NSK_OK;
}

static int conv_wgrad_impl(const nsk_conv_desc_t *desc, int groups, const void *x, const void *dy, float *dw,
                           int accumulate, void *workspace, size_t workspace_bytes, void *stream,
                           const float *act = nullptr, bool partial = false)   // partial: dw takes the partial sums
{
    ConvGeo g;
    NSK_TRY(conv_geometry(desc, &g, true));
    NSK_TRY(check_groups(g, groups));
    if (!x || !dy || !dw) return NSK_ERR_NULL;
    if (accumulate != 0 && accumulate != 1) return NSK_ERR_BAD_DESC;
    if (misaligned(x) || misaligned(dy) || misaligned(dw)) return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_act(g, groups, act));
    const ConvPlan p = plan_within(g, NSK_PASS_WGRAD, groups, act != nullptr, workspace, workspace_bytes);
    const int cg = g.C / groups, kg = g.K / groups;
    if (partial && !reduces_with_others(g, p)) return NSK_ERR_UNSUPPORTED;
    if (!partial) NSK_TRY(check_ws(workspace, workspace_bytes, p.total));
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    if (act && !p.act_fused) {   // the kernel for this layer does not apply the activation on load
        NSK_TRY(launch_bn_act(input_as_bn(g), x, act, ws + p.act_tmp, st));
        x = ws + p.act_tmp;
        if (p.stem) ws += align_up(g.x_elems * g.es);
    }
    const bool nchw = g.layout == NSK_NCHW;
    if (p.stem) return stem_wgrad(g, x, dy, dw, accumulate, ws, st);
    const void *xs = x, *dys = dy;
    const ConvGeo &gp = p.geo;
    const bool pad_c = gp.C != g.C, pad_k = gp.K != g.K;
    if (nchw) {
        NSK_TRY(launch_nchw_to_nhwc(g.dtype, x, ws + p.act_in, g.N, g.C, g.H, g.W, gp.C, st));
        NSK_TRY(launch_nchw_to_nhwc(g.dtype, dy, ws + p.act_in2, g.N, g.K, g.P, g.Q, gp.K, st));
    } else {
        if (pad_c) NSK_TRY(launch_pad_channels(g.dtype, x, ws + p.act_in, (long)g.N * g.H * g.W, g.C, gp.C, st));
        if (pad_k) NSK_TRY(launch_pad_channels(g.dtype, dy, ws + p.act_in2, (long)g.N * g.P * g.Q, g.K, gp.K, st));
    }
    if (nchw || pad_c) xs = ws + p.act_in;
    if (nchw || pad_k) dys = ws + p.act_in2;
    WgradArgs a{};
    a.x = xs; a.dy = dys; a.part = partial ? dw : (float *)(ws + p.part);
    wgrad_geometry(gp, &a);
    a.rows_per_split = p.rows_per_split;
    a.splits = p.splits;
    if (groups > 1) {   // `groups` problems of cg x kg channels; their partial sums stack to [splits][K][taps * cg]
        a.groups = groups;
        a.ldx = g.C;
        a.ldy = g.K;
        a.C = cg;
        a.K = kg;
    }
    if (p.pipe && groups <= 1) {
        a.groups = 1;
        a.ldx = gp.C;
        a.ldy = gp.K;
    }
    if (p.pipe && p.splits == 1 && !nchw && !accumulate && !pad_c && !pad_k) {   // one partial sum in the order of dw: it is the result
        a.part = dw;
        return launch_wgrad_pipe(g.dtype, a, st);
    }
    if (p.act_fused)
        NSK_TRY(launch_rows32_f32_act(a, act, st));
    else if (p.halo)
        NSK_TRY(launch_wgrad_halo64(a, st));
    else if (p.pipe)
        NSK_TRY(launch_wgrad_pipe(g.dtype, a, st));
    else if (p.grouped8)
        NSK_TRY(launch_grouped8_wgrad(a, st));
    else if (p.narrow)
        NSK_TRY(launch_narrow_wgrad(a, st));
    else
        NSK_TRY(launch_wgrad(g.dtype, a, st));
    if (partial) return NSK_OK;
    const long RS = (long)g.R * g.S;
    if (nchw)
        NSK_TRY(launch_wgrad_reduce(a.part, dw, p.splits, g.K, gp.K, a.ntaps, cg, gp.C / groups, (long)cg * RS, 1L, RS, accumulate, st));
    else
        NSK_TRY(launch_wgrad_reduce(a.part, dw, p.splits, g.K, gp.K, a.ntaps, cg, gp.C / groups, RS * cg, (long)cg, 1L, accumulate, st));
    return NSK_OK;
}

int nsk_conv2d_dgrad(const nsk_conv_desc_t *desc, const void *dy, const void *w, void *dx, int accumulate,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    return conv_dgrad_impl(desc, 1, dy, w, dx, accumulate, workspace, workspace_bytes, stream);
}

int nsk_conv2d_wgrad(const nsk_conv_desc_t *desc, const void *x, const void *dy, float *dw, int accumulate,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    return conv_wgrad_impl(desc, 1, x, dy, dw, accumulate, workspace, workspace_bytes, stream);
}

size_t nsk_conv2d_packed_filter_bytes(const nsk_conv_desc_t *desc)
{
    ConvGeo g;
    if (conv_geometry(desc, &g, true) != NSK_OK || !packs_with_others(g)) return 0;
    return align_up(g.w_elems * g.es + 256 * (size_t)g.sh * g.sw);
}

int nsk_conv2d_pack_filters(int count, const nsk_conv_item_t *items, void *stream)
{
    if (count < 0) return NSK_ERR_BAD_DESC;
    if (count > 0 && !items) return NSK_ERR_NULL;
    try {
        std::vector<PackItem> of[2];   // by type
        for (int i = 0; i < count; ++i) {
            if (!items[i].desc || !items[i].src || !items[i].dst) return NSK_ERR_NULL;
            // (stand-ins for the tensors that a packing does not read)
            NSK_TRY(conv_dgrad_impl(items[i].desc, 1, items[i].dst, items[i].src, items[i].dst, 0, nullptr, 0, stream, items[i].dst,
                                    &of[items[i].desc->dtype == NSK_BF16]));
        }
        for (int t = 0; t < 2; ++t) NSK_TRY(launch_pack_many(t ? NSK_BF16 : NSK_F32, of[t].data(), (int)of[t].size(), (hipStream_t)stream));
    } catch (const std::bad_alloc &) {
        return NSK_ERR_UNSUPPORTED;
    }
    return NSK_OK;
}

int nsk_conv2d_dgrad_packed(const nsk_conv_desc_t *desc, const void *dy, const void *packed, void *dx, int accumulate,
                            void *stream)
{
    if (!packed) return NSK_ERR_NULL;
    return conv_dgrad_impl(desc, 1, dy, packed, dx, accumulate, nullptr, 0, stream, const_cast<void *>(packed));
}

size_t nsk_conv2d_wgrad_partial_bytes(const nsk_conv_desc_t *desc)
{
    ConvGeo g;
    if (conv_geometry(desc, &g, true) != NSK_OK) return 0;
    const ConvPlan p = plan_conv(g, NSK_PASS_WGRAD);
    return reduces_with_others(g, p) ? (size_t)p.splits * g.w_elems * sizeof(float) : 0;
}

int nsk_conv2d_wgrad_partial(const nsk_conv_desc_t *desc, const void *x, const void *dy, float *partial, void *stream)
{
    return conv_wgrad_impl(desc, 1, x, dy, partial, 0, nullptr, 0, stream, nullptr, true);
}

int nsk_conv2d_wgrad_reduce(int count, const nsk_conv_item_t *items, int accumulate, void *stream)
{
    if (count < 0 || (accumulate != 0 && accumulate != 1)) return NSK_ERR_BAD_DESC;
    if (count > 0 && !items) return NSK_ERR_NULL;
    try {
        std::vector<ReduceItem> all;
        for (int i = 0; i < count; ++i) {
            ConvGeo g;
            NSK_TRY(conv_geometry(items[i].desc, &g, true));
            if (!items[i].src || !items[i].dst) return NSK_ERR_NULL;
            if (misaligned(items[i].src) || misaligned(items[i].dst)) return NSK_ERR_ALIGNMENT;
            const ConvPlan p = plan_conv(g, NSK_PASS_WGRAD);
            if (!reduces_with_others(g, p)) return NSK_ERR_UNSUPPORTED;
            all.push_back({(const float *)items[i].src, (float *)items[i].dst, p.splits, (int)g.w_elems, 0, 0});
        }
        return launch_wgrad_reduce_many(all.data(), (int)all.size(), accumulate, (hipStream_t)stream);
    } catch (const std::bad_alloc &) {
        return NSK_ERR_UNSUPPORTED;
    }
}

int nsk_conv2d_wgrad_act(const nsk_conv_desc_t *desc, const void *x, const float *coeffs, const void *dy, float *dw,
                         int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!coeffs) return NSK_ERR_NULL;
    return conv_wgrad_impl(desc, 1, x, dy, dw, accumulate, workspace, workspace_bytes, stream, coeffs);
}

size_t nsk_conv2d_grouped_workspace_bytes(const nsk_conv_desc_t *desc, int groups, int pass)
{
    ConvGeo g;
    if (pass < NSK_PASS_FWD || pass > NSK_PASS_WGRAD) return 0;
    if (conv_geometry(desc, &g, true) != NSK_OK || check_groups(g, groups) != NSK_OK) return 0;
    return plan_conv(g, pass, groups).total;
}

int nsk_conv2d_grouped_fwd(const nsk_conv_desc_t *desc, int groups, const void *x, const void *w, void *y,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    return conv_fwd_impl(desc, groups, x, w, y, nullptr, workspace, workspace_bytes, stream);
}

int nsk_conv2d_grouped_dgrad(const nsk_conv_desc_t *desc, int groups, const void *dy, const void *w, void *dx,
                             int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    return conv_dgrad_impl(desc, groups, dy, w, dx, accumulate, workspace, workspace_bytes, stream);
}

int nsk_conv2d_grouped_wgrad(const nsk_conv_desc_t *desc, int groups, const void *x, const void *dy, float *dw,
                             int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    return conv_wgrad_impl(desc, groups, x, dy, dw, accumulate, workspace, workspace_bytes, stream);
}

size_t nsk_bn_workspace_bytes(const nsk_bn_desc_t *desc, int pass)
{
    if (pass != NSK_BN_FWD && pass != NSK_BN_BWD) return 0;
    if (bn_geometry(desc) != NSK_OK) return 0;
    const size_t G = (size_t)bn_partial_blocks(*desc);
    const size_t floats = align_up((2 * G * desc->C + 4 * (size_t)desc->C) * sizeof(float));
    return floats + (pass == NSK_BN_BWD ? align_up(bn_mask_bytes(*desc)) : 0);
}

int nsk_bn_relu_add_fwd(const nsk_bn_desc_t *desc, const void *x, const void *residual, const float *gamma,
                        const float *beta, void *out, float *save_mean, float *save_invstd, float *running_mean,
                        float *running_var, void *workspace, size_t workspace_bytes, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!x || !gamma || !beta || !out || !save_mean || !save_invstd) return NSK_ERR_NULL;
    if ((running_mean == nullptr) != (running_var == nullptr)) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(residual) || misaligned(out) || misaligned(gamma) || misaligned(beta) ||
        misaligned(save_mean) || misaligned(save_invstd) || misaligned(running_mean) || misaligned(running_var))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_FWD)));
    return launch_bn_fwd(*desc, x, residual, gamma, beta, out, save_mean, save_invstd, running_mean, running_var,
                         workspace, nullptr, nullptr, 0, (hipStream_t)stream);
}

// ---- nsk_bn_relu_add_fwd for callers that cannot allocate: the partial sums live in a file-scope device array.
// The array's name is a host-side stand-in, not a device address: host code only ever uses the address that
// hipGetSymbolAddress returns for the current device (each GPU holds its own copy at its own address).
#define NSK_STATIC_SCRATCH_BYTES (8u << 20)
static __device__ __align__(256) unsigned char scratch[NSK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void **ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        nsk::set_last_hip_error(e);
        return NSK_ERR_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return NSK_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            nsk::set_last_hip_error(e);
            return NSK_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return NSK_OK;
}
}  // namespace

size_t nsk_static_scratch_bytes(void) { return NSK_STATIC_SCRATCH_BYTES; }

int nsk_bn_relu_add_fwd_static(const nsk_bn_desc_t *desc, const void *x, const void *residual, const float *gamma,
                               const float *beta, void *out, float *save_mean, float *save_invstd,
                               float *running_mean, float *running_var, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!x || !gamma || !beta || !out || !save_mean || !save_invstd) return NSK_ERR_NULL;
    if ((running_mean == nullptr) != (running_var == nullptr)) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(residual) || misaligned(out) || misaligned(gamma) || misaligned(beta) ||
        misaligned(save_mean) || misaligned(save_invstd) || misaligned(running_mean) || misaligned(running_var))
        return NSK_ERR_ALIGNMENT;
    // the partial sums of this descriptor must fit the static array (checked before any HIP call)
    if (nsk_bn_workspace_bytes(desc, NSK_BN_FWD) > NSK_STATIC_SCRATCH_BYTES) return NSK_ERR_WORKSPACE;
    void *ws = nullptr;
    NSK_TRY(static_scratch(&ws));
    // every partial sum the finalize kernel reads is written by the reduction of the same call: nothing to clear
    return launch_bn_fwd(*desc, x, residual, gamma, beta, out, save_mean, save_invstd, running_mean, running_var, ws,
                         nullptr, nullptr, 0, (hipStream_t)stream);
}

// ---- batch-norm + ReLU applied by the CONSUMERS of a convolution's raw output (the normalised activation is never stored)
int nsk_bn_fwd_coeffs(const nsk_bn_desc_t *desc, const float *gamma, const float *beta, const float *stats,
                      int stats_rows, float *save_mean, float *save_invstd, float *running_mean, float *running_var,
                      float *coeffs, void *workspace, size_t workspace_bytes, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!gamma || !beta || !stats || !save_mean || !save_invstd || !coeffs) return NSK_ERR_NULL;
    if (stats_rows < 1) return NSK_ERR_BAD_DESC;
    if ((running_mean == nullptr) != (running_var == nullptr)) return NSK_ERR_NULL;
    if (misaligned(gamma) || misaligned(beta) || misaligned(stats) || misaligned(save_mean) || misaligned(save_invstd) ||
        misaligned(running_mean) || misaligned(running_var) || misaligned(coeffs))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_FWD)));
    return launch_bn_coeffs(*desc, gamma, beta, stats, stats_rows, save_mean, save_invstd, running_mean, running_var,
                            coeffs, workspace, (hipStream_t)stream);
}

int nsk_conv2d_act_supported(const nsk_conv_desc_t *desc)
{
    ConvGeo g;
    if (conv_geometry(desc, &g, true) != NSK_OK) return 0;
    return g.layout == NSK_NHWC && bn_act_supported(input_as_bn(g)) ? 1 : 0;
}

size_t nsk_conv2d_act_workspace_bytes(const nsk_conv_desc_t *desc, int pass)
{
    ConvGeo g;
    if (pass != NSK_PASS_FWD && pass != NSK_PASS_WGRAD) return 0;
    if (conv_geometry(desc, &g, true) != NSK_OK) return 0;
    if (g.layout != NSK_NHWC || !bn_act_supported(input_as_bn(g))) return 0;
    return plan_conv(g, pass, 1, true).total;
}

int nsk_conv2d_fwd_act(const nsk_conv_desc_t *desc, const void *x, const float *coeffs, const void *w, void *y,
                       float *stats, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!coeffs) return NSK_ERR_NULL;
    if (misaligned(stats)) return NSK_ERR_ALIGNMENT;
    return conv_fwd_impl(desc, 1, x, w, y, stats, workspace, workspace_bytes, stream, coeffs);
}

int nsk_bn_relu_bwd_act(const nsk_bn_desc_t *desc, const void *x, const float *coeffs, const void *dout,
                        const float *gamma, const float *save_mean, const float *save_invstd, void *dx, float *dgamma,
                        float *dbeta, void *workspace, size_t workspace_bytes, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!x || !coeffs || !dout || !gamma || !save_mean || !save_invstd || !dx || !dgamma || !dbeta) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(coeffs) || misaligned(dout) || misaligned(dx) || misaligned(gamma) ||
        misaligned(save_mean) || misaligned(save_invstd) || misaligned(dgamma) || misaligned(dbeta))
        return NSK_ERR_ALIGNMENT;
    if (!desc->relu || desc->layout != NSK_NHWC || !bn_act_supported(*desc)) return NSK_ERR_UNSUPPORTED;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_BWD)));
    return launch_bn_bwd(*desc, x, nullptr, dout, gamma, save_mean, save_invstd, dx, nullptr, dgamma, dbeta, workspace,
                         nullptr, (hipStream_t)stream, coeffs);
}

int nsk_bn_relu_add_bwd(const nsk_bn_desc_t *desc, const void *x, const void *out, const void *dout,
                        const float *gamma, const float *save_mean, const float *save_invstd, void *dx,
                        void *dresidual, float *dgamma, float *dbeta, void *workspace, size_t workspace_bytes,
                        void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!x || !dout || !gamma || !save_mean || !save_invstd || !dx || !dgamma || !dbeta) return NSK_ERR_NULL;
    if (desc->relu && !out) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(out) || misaligned(dout) || misaligned(dx) || misaligned(dresidual) ||
        misaligned(gamma) || misaligned(save_mean) || misaligned(save_invstd) || misaligned(dgamma) ||
        misaligned(dbeta))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_BWD)));
    return launch_bn_bwd(*desc, x, out, dout, gamma, save_mean, save_invstd, dx, dresidual, dgamma, dbeta, workspace,
                         nullptr, (hipStream_t)stream);
}

size_t nsk_bn_mask_bytes(const nsk_bn_desc_t *desc)
{
    if (bn_geometry(desc) != NSK_OK) return 0;
    return bn_mask_bytes(*desc);
}

int nsk_bn_relu_add_fwd_mask(const nsk_bn_desc_t *desc, const void *x, const void *residual, const float *gamma,
                             const float *beta, void *out, unsigned char *relu_mask, float *save_mean,
                             float *save_invstd, float *running_mean, float *running_var, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (bn_mask_bytes(*desc) == 0) return NSK_ERR_UNSUPPORTED;
    if (!x || !gamma || !beta || !out || !relu_mask || !save_mean || !save_invstd) return NSK_ERR_NULL;
    if ((running_mean == nullptr) != (running_var == nullptr)) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(residual) || misaligned(out) || misaligned(relu_mask) || misaligned(gamma) ||
        misaligned(beta) || misaligned(save_mean) || misaligned(save_invstd) || misaligned(running_mean) ||
        misaligned(running_var))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_FWD)));
    return launch_bn_fwd(*desc, x, residual, gamma, beta, out, save_mean, save_invstd, running_mean, running_var,
                         workspace, relu_mask, nullptr, 0, (hipStream_t)stream);
}

int nsk_bn_relu_add_fwd_stats(const nsk_bn_desc_t *desc, const void *x, const void *residual, const float *gamma,
                              const float *beta, void *out, unsigned char *relu_mask, float *save_mean,
                              float *save_invstd, float *running_mean, float *running_var, const float *stats,
                              int stats_rows, void *workspace, size_t workspace_bytes, void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (!x || !gamma || !beta || !out || !save_mean || !save_invstd || !stats) return NSK_ERR_NULL;
    if (stats_rows < 1) return NSK_ERR_BAD_DESC;
    if (relu_mask && bn_mask_bytes(*desc) == 0) return NSK_ERR_UNSUPPORTED;
    if ((running_mean == nullptr) != (running_var == nullptr)) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(residual) || misaligned(out) || misaligned(relu_mask) || misaligned(gamma) ||
        misaligned(beta) || misaligned(save_mean) || misaligned(save_invstd) || misaligned(running_mean) ||
        misaligned(running_var) || misaligned(stats))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_FWD)));
    return launch_bn_fwd(*desc, x, residual, gamma, beta, out, save_mean, save_invstd, running_mean, running_var,
                         workspace, relu_mask, stats, stats_rows, (hipStream_t)stream);
}

int nsk_bn_relu_add_bwd_mask(const nsk_bn_desc_t *desc, const void *x, const unsigned char *relu_mask, const void *dout,
                             const float *gamma, const float *save_mean, const float *save_invstd, void *dx,
                             void *dresidual, float *dgamma, float *dbeta, void *workspace, size_t workspace_bytes,
                             void *stream)
{
    NSK_TRY(bn_geometry(desc));
    if (bn_mask_bytes(*desc) == 0) return NSK_ERR_UNSUPPORTED;
    if (!x || !relu_mask || !dout || !gamma || !save_mean || !save_invstd || !dx || !dgamma || !dbeta) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(relu_mask) || misaligned(dout) || misaligned(dx) || misaligned(dresidual) ||
        misaligned(gamma) || misaligned(save_mean) || misaligned(save_invstd) || misaligned(dgamma) || misaligned(dbeta))
        return NSK_ERR_ALIGNMENT;
    NSK_TRY(check_ws(workspace, workspace_bytes, nsk_bn_workspace_bytes(desc, NSK_BN_BWD)));
    return launch_bn_bwd(*desc, x, nullptr, dout, gamma, save_mean, save_invstd, dx, dresidual, dgamma, dbeta, workspace,
                         relu_mask, (hipStream_t)stream);
}

int nsk_maxpool2d_out_dims(const nsk_pool_desc_t *desc, int *P, int *Q)
{
    if (!desc || !P || !Q) return NSK_ERR_NULL;
    int p, q;
    NSK_TRY(pool_geometry(desc, &p, &q));
    *P = p;
    *Q = q;
    return NSK_OK;
}

int nsk_maxpool2d_fwd(const nsk_pool_desc_t *desc, const void *x, void *y, signed char *idx, void *stream)
{
    int P, Q;
    NSK_TRY(pool_geometry(desc, &P, &Q));
    if (P < 1 || Q < 1) return NSK_ERR_BAD_DESC;
    if (!x || !y || !idx) return NSK_ERR_NULL;
    if (misaligned(x) || misaligned(y) || misaligned(idx)) return NSK_ERR_ALIGNMENT;
    return launch_maxpool_fwd(*desc, P, Q, x, y, idx, (hipStream_t)stream);
}

int nsk_maxpool2d_bwd(const nsk_pool_desc_t *desc, const void *dy, const signed char *idx, void *dx, void *stream)
{
    int P, Q;
    NSK_TRY(pool_geometry(desc, &P, &Q));
    if (P < 1 || Q < 1) return NSK_ERR_BAD_DESC;
    if (!dy || !idx || !dx) return NSK_ERR_NULL;
    if (misaligned(dy) || misaligned(idx) || misaligned(dx)) return NSK_ERR_ALIGNMENT;
    return launch_maxpool_bwd(*desc, P, Q, dy, idx, dx, (hipStream_t)stream);
}

}  // extern "C"
