"""Layers whose channel counts are not whole 16-byte vectors: the operands are copied with zero channels up to the next whole
vector and the kernels for whole vectors run.  All passes, both layouts, old values added, statistics, against the oracle and
against the element-wise kernels (the copies switched off); values that are not finite stay where they reach."""
import ctypes

import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, to_gpu, to_host, torch_dtype

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad, dilation
SHAPES = [
    (2, 5, 6, 7, 9, 3, 3, 1, 1, 1),            # fewest channels that are copied in bf16, odd bytes per row
    (2, 7, 6, 7, 9, 3, 3, 1, 1, 1),            # ... in fp32
    (1, 12, 1, 1, 20, 1, 1, 1, 0, 1),          # one pixel; bf16 rows of 24 and 40 bytes
    (3, 100, 9, 11, 36, 3, 3, 1, 1, 1),
    (2, 62, 14, 10, 16, 3, 3, 2, 1, 1),        # C alone; bf16 rows of 4-byte units
    (2, 16, 13, 9, 60, 3, 3, 2, 1, 1),         # K alone, four classes backward
    (4, 60, 16, 16, 60, 3, 3, 1, 1, 1),        # becomes a 64 -> 64 layer
    (3, 20, 10, 8, 44, 1, 1, 2, 0, 1),         # classes without a tap
    (2, 13, 12, 20, 70, 2, 3, (1, 2), (0, 1), (2, 1)),
    (2, 9, 10, 9, 11, 3, 3, 3, 1, 1),          # nine classes: launched one by one
]


@pytest.mark.parametrize("layout", [B.NSK_NHWC, B.NSK_NCHW], ids=["nhwc", "nchw"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_padded_channels(i, dtype, layout, nsk_env):
    N, C, H, W, K, R, S, st, pd, dl = SHAPES[i]
    print(f"channels not in whole vectors, {SHAPES[i]} {dtype} layout {layout}", flush=True)
    tol = TOL[dtype]
    x = on_grid(gen.normal(990 + i, 0, (N, C, H, W)), dtype)
    w = on_grid(gen.he_normal(990 + i, 1, (K, C, R, S)), dtype)
    P, Q = oracle.conv2d_out_dims(x.shape, w.shape, st, pd, dl)
    dy = on_grid(gen.normal(990 + i, 2, (N, K, P, Q)), dtype)
    old = on_grid(gen.normal(990 + i, 3, x.shape), dtype)
    gx, gw, gdy = (to_gpu(a, dtype, layout) for a in (x, w, dy))
    wshape = (K, R, S, C) if layout == B.NSK_NHWC else (K, C, R, S)

    def passes():
        ws, out = B.Workspace(), {}
        y, ok = guarded(gdy.shape, torch_dtype(dtype))
        _, stats = B.conv2d_fwd_stats(gx, gw, st, pd, dl, layout, out=y, ws=ws)
        torch.cuda.synchronize()
        ok()
        out["y"], sums = to_host(y, layout), stats.double().sum(1).cpu().numpy()
        n = N * P * Q      # float sums of at most n stored values: see the bars of the pipelined kernel's test
        assert np.allclose(sums[0], out["y"].sum((0, 2, 3)), rtol=0, atol=1e-6 * n * np.abs(out["y"]).max())
        assert np.allclose(sums[1], (out["y"] ** 2).sum((0, 2, 3)), rtol=1e-5, atol=1e-6)
        plain = B.conv2d_fwd(gx, gw, st, pd, dl, layout, ws=ws)
        assert max_rel_err(to_host(plain, layout), out["y"]) <= tol     # (may be another kernel)
        for name, accumulate in (("dx", False), ("dx_old", True)):
            dx, ok = guarded(gx.shape, torch_dtype(dtype))
            if accumulate:
                dx.copy_(to_gpu(old, dtype, layout))
            B.conv2d_dgrad(gdy, gw, x.shape, st, pd, dl, layout, out=dx, accumulate=accumulate, ws=ws)
            torch.cuda.synchronize()
            ok()
            out[name] = to_host(dx, layout)
        dw, ok = guarded(wshape, torch.float32)
        B.conv2d_wgrad(gx, gdy, w.shape, st, pd, dl, layout, out=dw, ws=ws)
        torch.cuda.synchronize()
        ok()
        out["dw"] = to_host(dw, layout)
        first = dw.clone()
        B.conv2d_wgrad(gx, gdy, w.shape, st, pd, dl, layout, out=dw, accumulate=True, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(dw, first + first)
        return out

    got = passes()
    assert max_rel_err(got["y"], oracle.conv2d_fwd(x, w, st, pd, dl)) <= tol
    want = oracle.conv2d_dgrad(dy, w, x.shape, st, pd, dl)
    assert max_rel_err(got["dx"], want) <= tol
    assert max_rel_err(got["dx_old"], want + old) <= tol
    assert max_rel_err(got["dw"], oracle.conv2d_wgrad(x, dy, w.shape, st, pd, dl)) <= TOL["f32"]   # exact products, float sums
    nsk_env("NSK_NO_PAD", "1")
    general = passes()
    for name in got:
        assert max_rel_err(got[name], general[name]) <= (TOL["f32"] if name == "dw" else tol)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_values_that_are_not_finite(dtype, nsk_env):
    N, C, H, W, K = 2, 13, 6, 7, 11
    x, w = gen.normal(999, 0, (N, C, H, W)).astype(np.float32), gen.he_normal(999, 1, (K, C, 3, 3)).astype(np.float32)
    dy = gen.normal(999, 2, (N, K, H, W)).astype(np.float32)
    x[0, 12, 2, 3], x[1, 0, 5, 6], dy[1, 10, 0, 0], dy[0, 4, 3, 3] = np.inf, np.nan, -np.inf, np.nan   # last and first channels of a pixel
    lay = B.NSK_NHWC
    gx, gw, gdy = (to_gpu(a, dtype, lay) for a in (x, w, dy))

    def passes():
        return [B.conv2d_fwd(gx, gw, 1, 1), B.conv2d_dgrad(gdy, gw, x.shape, 1, 1), B.conv2d_wgrad(gx, gdy, w.shape, 1, 1)]

    got = passes()
    nsk_env("NSK_NO_PAD", "1")
    for a, b in zip(got, passes()):
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        assert torch.equal(torch.isinf(a), torch.isinf(b)) and not torch.isfinite(a).all() and torch.isfinite(a).any()


@pytest.mark.parametrize("layout", [B.NSK_NHWC, B.NSK_NCHW], ids=["nhwc", "nchw"])
@pytest.mark.parametrize("dtype,C,K", [("bf16", 20, 36), ("bf16", 13, 24), ("f32", 30, 10), ("f32", 9, 7)])
def test_a_workspace_without_room_for_the_copies(dtype, C, K, layout, nsk_env):
    """The layer then runs on the operands as they lie, with what that needs: nothing at all for a forward pass in NHWC."""
    N, H, W, t = 2, 9, 11, torch_dtype(dtype)
    x, dy = (on_grid(gen.normal(996, k, (N, c, H, W)), dtype) for k, c in ((0, C), (2, K)))
    w = on_grid(gen.he_normal(996, 1, (K, C, 3, 3)), dtype)
    gx, gw, gdy = (to_gpu(a, dtype, layout) for a in (x, w, dy))
    d = B.conv_desc((N, C, H, W), (K, 3, 3), 1, 1, 1, B._dtype_code(gx), layout)
    ref, L = ctypes.byref(d), B.lib()
    full = [L.nsk_conv2d_workspace_bytes(ref, p) for p in range(3)]
    rows = int(L.nsk_conv2d_stats_rows(ref))
    nsk_env("NSK_NO_PAD", "1")
    least = [L.nsk_conv2d_workspace_bytes(ref, p) for p in range(3)]
    nsk_env("NSK_NO_PAD", None)
    assert [L.nsk_conv2d_workspace_bytes(ref, p) for p in range(3)] == full
    assert least[0] < full[0] and (layout == B.NSK_NCHW or least[0] == 0)
    ws = torch.empty(max(least + [1]), dtype=torch.uint8, device="cuda:0")
    at = lambda p: (ws.data_ptr() if least[p] else None, least[p])
    stream = torch.cuda.current_stream().cuda_stream
    y, check = guarded(gdy.shape, t)
    stats, check_stats = guarded((2, rows, K), torch.float32)
    assert L.nsk_conv2d_fwd(ref, gx.data_ptr(), gw.data_ptr(), y.data_ptr(), *at(0), stream) == B.NSK_OK
    first = y.clone()
    y.zero_()
    stats.fill_(float("nan"))
    assert L.nsk_conv2d_fwd_stats(ref, gx.data_ptr(), gw.data_ptr(), y.data_ptr(), stats.data_ptr(), *at(0), stream) == B.NSK_OK
    dx, dw = torch.empty_like(gx), torch.empty(gw.shape, device="cuda:0")
    assert L.nsk_conv2d_dgrad(ref, gdy.data_ptr(), gw.data_ptr(), dx.data_ptr(), 0, *at(1), stream) == B.NSK_OK
    assert L.nsk_conv2d_wgrad(ref, gx.data_ptr(), gdy.data_ptr(), dw.data_ptr(), 0, *at(2), stream) == B.NSK_OK
    torch.cuda.synchronize()
    check()
    check_stats()
    assert torch.equal(y, first)
    got = to_host(y, layout)
    assert max_rel_err(got, oracle.conv2d_fwd(x, w, 1, 1, 1)) <= TOL[dtype]
    # float sums of at most 198 values in every row: 198 roundings of the largest partial sum
    sums = stats.double().sum(1).cpu().numpy()
    assert np.abs(sums[0] - got.sum((0, 2, 3))).max() <= 198 * 2.0 ** -24 * np.abs(got).sum((0, 2, 3)).max()
    assert np.abs(sums[1] - (got ** 2).sum((0, 2, 3))).max() <= 198 * 2.0 ** -24 * (got ** 2).sum((0, 2, 3)).max()
    assert max_rel_err(to_host(dx, layout), oracle.conv2d_dgrad(dy, w, x.shape, 1, 1, 1)) <= TOL[dtype]
    assert max_rel_err(to_host(dw, layout), oracle.conv2d_wgrad(x, dy, w.shape, 1, 1, 1)) <= TOL["f32"]
    for p in (0, 1, 2):                 # less than that is refused as ever
        if least[p]:
            args = [(gx, gw, y), (gdy, gw, dx), (gx, gdy, dw)][p]
            call = [L.nsk_conv2d_fwd, L.nsk_conv2d_dgrad, L.nsk_conv2d_wgrad][p]
            mid = () if p == 0 else (0,)
            assert call(ref, *(a.data_ptr() for a in args), *mid, ws.data_ptr(), least[p] - 1, stream) == B.NSK_ERR_WORKSPACE
