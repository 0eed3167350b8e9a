"""The pipelined backward-weight kernel, every tile shape of it, where a tile can go wrong: fewer k-tiles than stages and every
remainder of them, one and several splits, ragged rows and columns, stride, dilation, images of one pixel, groups; and the
bf16 64 -> 64 kernel on problems that are below the size from which it is chosen."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, to_gpu, to_host

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad, dilation; a k-tile is 64 (bf16) or 32 (f32) output pixels
SHAPES = [
    (1, 8, 1, 1, 8, 1, 1, 1, 0, 1),            # one pixel
    (50, 24, 1, 1, 72, 1, 1, 1, 0, 1),         # images of one pixel (a fully connected layer), one ragged k-tile
    (1, 16, 9, 9, 40, 3, 3, 1, 1, 1),          # two (three) k-tiles
    (3, 40, 13, 11, 136, 3, 3, 1, 1, 1),       # 429 pixels: 7 (14) k-tiles, images change inside them
    (2, 64, 21, 18, 64, 3, 3, 2, 1, 1),        # stride 2
    (2, 24, 12, 20, 200, 2, 3, (1, 2), (0, 1), (2, 1)),
    (6, 8, 40, 41, 8, 7, 7, 1, 3, 1),          # 9840 pixels: chains of k-tiles are banked; several splits
]


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_every_tile(i, dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    nsk_env("NSK_NO_HALO", "1")
    N, C, H, W, K, R, S, st, pd, dl = SHAPES[i]
    print(f"pipelined backward-weight, shape {SHAPES[i]} {dtype} tile {tile}", flush=True)
    x = on_grid(gen.normal(960 + i, 0, (N, C, H, W)), dtype)
    P, Q = oracle.conv2d_out_dims(x.shape, (K, C, R, S), st, pd, dl)
    dy = on_grid(gen.normal(960 + i, 2, (N, K, P, Q)), dtype)
    want = oracle.conv2d_wgrad(x, dy, (K, C, R, S), st, pd, dl)
    for lay in (B.NSK_NHWC, B.NSK_NCHW):
        gx, gdy, ws = to_gpu(x, dtype, lay), to_gpu(dy, dtype, lay), B.Workspace()
        shape = (K, R, S, C) if lay == B.NSK_NHWC else (K, C, R, S)
        dw, check = guarded(shape, torch.float32)
        B.conv2d_wgrad(gx, gdy, (K, C, R, S), st, pd, dl, lay, out=dw, ws=ws)
        torch.cuda.synchronize()
        check()
        first = dw.clone()
        assert max_rel_err(to_host(dw, lay), want) <= TOL["f32"]     # float sums of exact products in both types
        B.conv2d_wgrad(gx, gdy, (K, C, R, S), st, pd, dl, lay, out=dw, accumulate=True, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(dw, first + first)                         # the same sum, added to the one it already holds


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_every_tile_grouped(dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, cg, kg, G, H, W = 2, 16, 24, 3, 19, 13
    x = on_grid(gen.normal(980, 0, (N, G * cg, H, W)), dtype)
    dy = on_grid(gen.normal(980, 2, (N, G * kg, H, W)), dtype)
    dw = to_host(B.conv2d_grouped_wgrad(to_gpu(x, dtype, B.NSK_NHWC), to_gpu(dy, dtype, B.NSK_NHWC), (G * kg, cg, 3, 3), G, 1, 1), B.NSK_NHWC)
    for g in range(G):
        c, k = slice(g * cg, (g + 1) * cg), slice(g * kg, (g + 1) * kg)
        assert max_rel_err(dw[k], oracle.conv2d_wgrad(x[:, c], dy[:, k], (kg, cg, 3, 3), 1, 1, 1)) <= TOL["f32"]


# A float sum of n terms of either sign, added one after the other, is off by about 2.5e-8 * sqrt(n / 2) of its size (2.5e-8: the
# rms of one rounding).  fp32: chains of at most 128 pixels 2.0e-7, with the few sums of chains and splits behind them 2.2e-7;
# bf16: 8 products of 16 pixels, four roundings in each, 1.0e-7, 16 products in splits of more than 16 k-tiles (the last), 1.4e-7.
@pytest.mark.parametrize("dtype,bar,N,C,H,K,R,stride", [("f32", 1.9e-7, 8, 16, 32, 16, 3, 1),       # 64 splits of 128 pixels: chains of 64, 1.4e-7
                                                        ("f32", 2.3e-7, 3, 744, 24, 744, 1, 2), ("f32", 2.3e-7, 7, 48, 17, 808, 3, 1),
                                                        ("bf16", 1.05e-7, 3, 416, 25, 416, 1, 1), ("bf16", 1.5e-7, 4, 48, 65, 240, 3, 1)])
def test_error_does_not_grow_with_the_split(dtype, bar, N, C, H, K, R, stride):
    g = torch.Generator(device="cuda").manual_seed(11)
    P, pad = (H - 1) // stride + 1, R // 2
    d = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.randn((N, H, H, C), generator=g, device="cuda").to(d)
    dy = torch.randn((N, P, P, K), generator=g, device="cuda").to(d)
    dw = B.conv2d_wgrad(x, dy, (K, C, R, R), stride, pad).double()
    xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    for r in range(R):
        for s in range(R):
            xs = xp[:, r:r + (P - 1) * stride + 1:stride, s:s + (P - 1) * stride + 1:stride].reshape(-1, C)
            want = dy.double().reshape(-1, K).t() @ xs
            assert float((dw[:, r, s] - want).norm() / want.norm()) <= bar, (r, s)


# (fp32 layers of these channels run on the pipelined kernel)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 7, 9), (3, 20, 20), (2, 16, 32), (5, 6, 66)])
def test_64_to_64_layers_below_the_size_of_their_kernel(shape, dtype, nsk_env):
    nsk_env("NSK_WH_MIN_ROWS", "1")
    N, H, W = shape
    x, dy = (on_grid(gen.normal(990, t, (N, 64, H, W)), dtype) for t in (0, 2))
    dw = B.conv2d_wgrad(to_gpu(x, dtype, B.NSK_NHWC), to_gpu(dy, dtype, B.NSK_NHWC), (64, 64, 3, 3), 1, 1)
    assert max_rel_err(to_host(dw, B.NSK_NHWC), oracle.conv2d_wgrad(x, dy, (64, 64, 3, 3), 1, 1, 1)) <= TOL["f32"]
