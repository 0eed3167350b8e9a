"""fp32 products on the bf16 matrix unit (three bf16 pieces a value): every tile shape that makes them at the edges of tiles and k-tiles,
their error against 64 bits, and operands that the pieces cannot hold, whose tiles are made again on the fp32 unit."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, to_gpu, to_host

pytestmark = pytest.mark.gpu

LAY = B.NSK_NHWC
# N, C, H, W, K, R, stride; a k-tile is 32 reduction indices, two groups of 16
SHAPES = [
    (1, 4, 5, 5, 4, 1, 1),         # a quarter of a group
    (2, 20, 9, 11, 36, 1, 1),      # one group and a quarter of the second
    (3, 24, 17, 13, 72, 3, 1),     # taps change inside k-tiles
    (2, 64, 14, 10, 132, 3, 2),    # strided classes, a column tile of four
    (5, 320, 7, 7, 264, 1, 1),     # ten k-tiles, three column tiles of 128
    (9, 16, 33, 31, 16, 3, 1),     # 9207 pixels: several splits and row tiles
]


@pytest.mark.parametrize("tile", range(1, 7))
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_every_tile(i, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K, R, st = SHAPES[i]
    print(f"pieces, shape {SHAPES[i]} tile {tile}", flush=True)
    x, w = gen.normal(1900 + i, 0, (N, C, H, W)), gen.he_normal(1900 + i, 1, (K, C, R, R))
    P, Q = oracle.conv2d_out_dims(x.shape, w.shape, st, R // 2, 1)
    dy, old = gen.normal(1900 + i, 2, (N, K, P, Q)), gen.normal(1900 + i, 3, x.shape)
    gx, gw, gdy, ws = to_gpu(x, "f32", LAY), to_gpu(w, "f32", LAY), to_gpu(dy, "f32", LAY), B.Workspace()
    for out, want, call in (
            (gdy, oracle.conv2d_fwd(x, w, st, R // 2, 1), lambda o: B.conv2d_fwd(gx, gw, st, R // 2, out=o, ws=ws)),
            (gx, oracle.conv2d_dgrad(dy, w, x.shape, st, R // 2, 1), lambda o: B.conv2d_dgrad(gdy, gw, x.shape, st, R // 2, out=o, ws=ws)),
            (gw, oracle.conv2d_wgrad(x, dy, w.shape, st, R // 2, 1), lambda o: B.conv2d_wgrad(gx, gdy, w.shape, st, R // 2, out=o, ws=ws))):
        got, check = guarded(out.shape, torch.float32)
        call(got)
        torch.cuda.synchronize()
        check()
        assert max_rel_err(to_host(got, LAY), want) <= TOL["f32"]
    dx = B.conv2d_dgrad(gdy, gw, x.shape, st, R // 2, out=to_gpu(old, "f32", LAY), accumulate=True, ws=ws)
    assert max_rel_err(to_host(dx, LAY), oracle.conv2d_dgrad(dy, w, x.shape, st, R // 2, 1) + old) <= TOL["f32"]


# What decayed filters and vanishing gradients come to: the last bits of either operand below what a bf16 can hold by itself (2^-133) from 2^-110
# on, subnormal floats at 2^-126.  The other operand is of ordinary size, and the results are floats; one tolerance for all passes.
@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("exponent", [-112, -120, -126])
def test_tiny_operands(exponent, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K = 2, 40, 12, 11, 72
    tiny = np.float32(2.0 ** exponent)
    x, w, dy = gen.normal(1960, 0, (N, C, H, W)), gen.he_normal(1960, 1, (K, C, 1, 1)), gen.normal(1960, 2, (N, K, H, W))
    calls = {
        "forward": (x, w, "nchw,kc->nkhw", lambda a, b: B.conv2d_fwd(a, b, 1, 0)),
        "backward-data": (dy, w, "nkhw,kc->nchw", lambda a, b: B.conv2d_dgrad(a, b, x.shape, 1, 0)),
        "backward-weight": (x, dy, "nchw,nkhw->kc", lambda a, b: B.conv2d_wgrad(a, b, w.shape, 1, 0)),
    }
    for name, (a, b, product, call) in calls.items():
        for a_, b_ in ((a * tiny, b), (a, b * tiny)):
            flat = [v[:, :, 0, 0] if v.shape[2:] == (1, 1) else v for v in (a_.astype(np.float64), b_.astype(np.float64))]
            want = np.einsum(product, *flat)
            got = to_host(call(to_gpu(a_, "f32", LAY), to_gpu(b_, "f32", LAY)), LAY).reshape(want.shape)
            assert np.max(np.abs(got - want)) <= 2e-6 * np.sqrt(np.mean(want ** 2)), (name, a_ is a)


# A sum with one product in it (one channel, one pixel, one output channel that is not zero), x and y from 1 to 2: the middle pieces are at most 2^-8
# and the last ones 2^-17, so leaving out the two products of a middle and a last one costs at most 2^-24, the rounding as much.  rms: 2.53e-8 of a
# rounding, and 2^-25 / 3 each for uniform pieces, halved by the mean of 1 / (xy)^2, 0.7e-8: 2.62e-8 in quadrature.
@pytest.mark.parametrize("tile", [1, 2, 3, 4])
def test_a_sum_of_one_product(tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K = 2, 36, 16, 16, 68
    r = np.random.default_rng(9)
    mantissas = lambda *shape: (r.integers(1 << 23, 1 << 24, shape) * 2.0 ** -23).astype(np.float32)
    x, w, dy = np.zeros((N, C, H, W), np.float32), mantissas(K, C, 1, 1), np.zeros((N, K, H, W), np.float32)
    n, h, v = np.meshgrid(np.arange(N), np.arange(H), np.arange(W), indexing="ij")
    x[n, (5 * n + 3 * h + v) % C, h, v] = mantissas(N, H, W)
    dy[n, (n + 7 * h + v) % K, h, v] = mantissas(N, H, W)
    x1, dy1 = np.zeros_like(x), np.zeros_like(dy)       # backward-weight: one pixel
    x1[1, :, 7, 9], dy1[1, :, 7, 9] = mantissas(C), mantissas(K)
    d = lambda a: a.astype(np.float64)
    for name, got, want in (
            ("forward", B.conv2d_fwd(to_gpu(x, "f32", LAY), to_gpu(w, "f32", LAY), 1, 0), np.einsum("nchw,kc->nkhw", d(x), d(w[:, :, 0, 0]))),
            ("backward-data", B.conv2d_dgrad(to_gpu(dy, "f32", LAY), to_gpu(w, "f32", LAY), x.shape, 1, 0), np.einsum("nkhw,kc->nchw", d(dy), d(w[:, :, 0, 0]))),
            ("backward-weight", B.conv2d_wgrad(to_gpu(x1, "f32", LAY), to_gpu(dy1, "f32", LAY), w.shape, 1, 0), np.einsum("nchw,nkhw->kc", d(x1), d(dy1)))):
        got = to_host(got, LAY).reshape(want.shape)
        off = ((got - want) / np.where(want == 0, 1, want))[want != 0]
        assert np.all(got[want == 0] == 0)
        assert np.max(np.abs(off)) <= 2.0 ** -23, (name, np.max(np.abs(off)))
        assert np.sqrt(np.mean(off ** 2)) <= 2.65e-8 * (1 + 2 / off.size ** 0.5), (name, np.sqrt(np.mean(off ** 2)))


# One rounding of a sum is 2.5e-8 (rms) of its size, n of them in a row 2.5e-8 * sqrt(n / 2).  A product of 16 indices rounds its large sum
# twice (eight indices at a time): 288 roundings for 2304 indices, 3.0e-7, and what the smaller products, the last additions and the splits add,
# below 0.8e-7, makes 3.1e-7 in quadrature; where two wavefronts share the reduction 144 of them, 2.3e-7.
@pytest.mark.parametrize("tile,bar", [(1, 2.3e-7), (2, 2.3e-7), (3, 3.1e-7), (4, 3.1e-7)])
def test_error_against_64_bits(tile, bar, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    g = torch.Generator().manual_seed(7)
    x, w = torch.randn(8, 256, 16, 16, generator=g), torch.randn(128, 256, 3, 3, generator=g) * 0.03
    dy = torch.randn(8, 128, 16, 16, generator=g)
    nhwc = lambda t: t.permute(0, 2, 3, 1).contiguous().cuda()
    rel = lambda got, want: float((got.permute(0, 3, 1, 2).cpu().double() - want).norm() / want.norm())
    y = B.conv2d_fwd(nhwc(x), nhwc(w), 1, 1)
    assert rel(y, torch.nn.functional.conv2d(x.double(), w.double(), padding=1)) <= bar
    dw = B.conv2d_wgrad(nhwc(x), nhwc(dy), tuple(w.shape), 1, 1)
    assert rel(dw, torch.nn.grad.conv2d_weight(x.double(), w.shape, dy.double(), padding=1)) <= bar


def _same(got, want, tol):
    """The same infinities and NaN; finite values to tol of the largest neighbour they could come from."""
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    if ok.any():
        scale = np.sqrt(np.mean(want[ok] ** 2))
        assert np.max(np.abs(got[ok] - want[ok])) <= tol * scale


@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("what", ["inf", "nan", "opposite", "largest", "large sums", "smallest"])
def test_operands_beyond_the_pieces(what, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K = 2, 40, 12, 11, 72
    x, w = gen.normal(1950, 0, (N, C, H, W)), gen.he_normal(1950, 1, (K, C, 1, 1))
    dy = gen.normal(1950, 2, (N, K, H, W))
    w[3, 5] = 0.0                      # an infinity times zero
    if what == "inf":
        x[1, 5, 3, 4] = np.inf
    elif what == "nan":
        x[0, 7, 11, 10] = np.nan
    elif what == "opposite":
        x[0, 5, 2, 2], x[0, 6, 2, 2] = np.inf, -np.inf
    elif what == "largest":            # above the largest bf16; products of 1/4 stay in range
        x[0, 1, 1, 1], w[:, 1] = np.float32(3.4e38), 0.25
        dy[0, :, 1, 1] = 0.25
    elif what == "large sums":         # 2^90, finite, but not times 2^48
        x, w, dy = x * np.float32(2.0 ** 60), w * np.float32(2.0 ** 30), dy * np.float32(2.0 ** 30)
    else:                              # the last pieces would lie below the smallest bf16
        x, dy = x * np.float32(2.0 ** -112), dy * np.float32(2.0 ** -112)
    x64, w64, dy64 = x.astype(np.float64), w[:, :, 0, 0].astype(np.float64), dy.astype(np.float64)
    gx, gw, gdy = (to_gpu(a, "f32", LAY) for a in (x, w, dy))
    f32 = np.finfo(np.float32).max
    clip = lambda a: np.where(np.abs(a) > f32, np.sign(a) * np.inf, a)
    with np.errstate(invalid="ignore", over="ignore"):
        y_want = clip(np.einsum("nchw,kc->nkhw", x64, w64))
        _same(to_host(B.conv2d_fwd(gx, gw, 1, 0), LAY), y_want, 2e-6)
        one = np.ones_like(dy64) if what == "smallest" else dy64      # (the product of both would not be a float)
        gone = to_gpu(one.astype(np.float32), "f32", LAY)
        dw_want = clip(np.einsum("nkhw,nchw->kc", one, x64))
        _same(to_host(B.conv2d_wgrad(gx, gone, w.shape, 1, 0), LAY)[:, :, 0, 0], dw_want, 2e-6 if what == "smallest" else 1e-5)
        if what in ("smallest", "large sums"):
            _same(to_host(B.conv2d_dgrad(gdy, gw, x.shape, 1, 0), LAY), np.einsum("nkhw,kc->nchw", dy64, w64), 2e-6)


# Backward-data that fetches its filter without a packing: up to eight k-tiles on the smallest tile; taps inside k-tiles, strided classes (and
# some without a tap), channel counts that are copied to whole vectors, one k-tile more (packed); the forced tile takes other problems too.
@pytest.mark.parametrize("tile", [None, "6"])
@pytest.mark.parametrize("N,C,H,W,K,R,S,st,pd", [(2, 16, 9, 11, 16, 3, 3, 1, 1), (1, 20, 12, 7, 28, 3, 3, 2, 1), (3, 36, 7, 7, 64, 1, 1, 2, 0), (2, 8, 10, 9, 4, 7, 7, 1, 3),
                                                 (1, 40, 6, 6, 256, 1, 1, 1, 0), (1, 40, 6, 6, 260, 1, 1, 1, 0), (2, 30, 8, 8, 22, 3, 3, 1, 1), (1, 12, 9, 9, 12, 2, 2, 2, 0)])
def test_filter_without_packing(N, C, H, W, K, R, S, st, pd, tile, nsk_env):
    if tile:
        nsk_env("NSK_IGEMM_TILE", tile)
    w = gen.he_normal(1970, 1, (K, C, R, S))
    P, Q = oracle.conv2d_out_dims((N, C, H, W), w.shape, st, pd, 1)
    dy, old = gen.normal(1970, 2, (N, K, P, Q)), gen.normal(1970, 3, (N, C, H, W))
    want = oracle.conv2d_dgrad(dy, w, (N, C, H, W), st, pd, 1)
    gw, gdy, gold = (to_gpu(a, "f32", LAY) for a in (w, dy, old))
    for accumulate in (False, True):
        dx, check = guarded(gold.shape, torch.float32)
        if accumulate:
            dx.copy_(gold)
        B.conv2d_dgrad(gdy, gw, (N, C, H, W), st, pd, out=dx, accumulate=accumulate)
        torch.cuda.synchronize()
        check()
        assert max_rel_err(to_host(dx, LAY), want + old if accumulate else want) <= TOL["f32"]
