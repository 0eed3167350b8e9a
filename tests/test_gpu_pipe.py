"""The pipelined implicit-GEMM kernel, every tile shape of it, where a tile can go wrong: fewer k-tiles than stages and
every remainder of them, several taps inside one k-tile, ragged rows and columns, strided classes, old values added,
statistics, groups.  The tile is forced through its test hook (which also keeps the other kernels out)."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, to_gpu, to_host, torch_dtype

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad, dilation; a k-tile is 64 (bf16) or 32 (f32) reduction indices
SHAPES = [
    (1, 8, 5, 5, 8, 1, 1, 1, 0, 1),            # one short k-tile, one tile
    (2, 40, 9, 11, 40, 1, 1, 1, 0, 1),         # one or two k-tiles, ragged on all sides
    (3, 24, 17, 13, 72, 3, 3, 1, 1, 1),        # 216 indices: taps change inside k-tiles, remainder of the stages
    (2, 64, 14, 10, 136, 3, 3, 2, 1, 1),       # stride 2: four classes in backward-data, 9 k-tiles
    (2, 16, 12, 20, 200, 2, 3, (1, 2), (0, 1), (2, 1)),   # four taps a k-tile, anisotropic
    (1, 8, 15, 15, 8, 7, 7, 1, 3, 1),          # 49 taps of 8 channels
    (5, 320, 7, 7, 264, 1, 1, 1, 0, 1),        # 5 k-tiles (bf16), 10 (f32), three column tiles of 128
]


TILES = [("f32", t) for t in range(1, 7)] + [("bf16", t) for t in range(1, 8)]


@pytest.mark.parametrize("dtype,tile", TILES)
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_every_tile(i, dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K, R, S, st, pd, dl = SHAPES[i]
    print(f"pipelined kernel, shape {SHAPES[i]} {dtype} tile {tile}", flush=True)
    tol, ws, lay = TOL[dtype], B.Workspace(), B.NSK_NHWC
    x = on_grid(gen.normal(900 + i, 0, (N, C, H, W)), dtype)
    w = on_grid(gen.he_normal(900 + i, 1, (K, C, R, S)), dtype)
    P, Q = oracle.conv2d_out_dims(x.shape, w.shape, st, pd, dl)
    dy = on_grid(gen.normal(900 + i, 2, (N, K, P, Q)), dtype)
    old = on_grid(gen.normal(900 + i, 3, x.shape), dtype)
    gx, gw, gdy = (to_gpu(a, dtype, lay) for a in (x, w, dy))

    y, check = guarded(gdy.shape, torch_dtype(dtype))
    _, stats = B.conv2d_fwd_stats(gx, gw, st, pd, dl, lay, out=y, ws=ws)
    torch.cuda.synchronize()
    check()
    got = to_host(y, lay)
    assert max_rel_err(got, oracle.conv2d_fwd(x, w, st, pd, dl)) <= tol
    # float sums of at most N*P*Q stored values of either sign: absolute bars of sqrt(n) roundings of the largest partial sum
    sums = stats.double().sum(1).cpu().numpy()
    n = N * P * Q
    assert np.allclose(sums[0], got.sum((0, 2, 3)), rtol=0, atol=1e-6 * n * np.abs(got).max())
    assert np.allclose(sums[1], (got ** 2).sum((0, 2, 3)), rtol=1e-5, atol=1e-6)

    want = oracle.conv2d_dgrad(dy, w, x.shape, st, pd, dl)
    for accumulate in (False, True):
        dx, check = guarded(gx.shape, torch_dtype(dtype))
        if accumulate:
            dx.copy_(to_gpu(old, dtype, lay))
        B.conv2d_dgrad(gdy, gw, x.shape, st, pd, dl, lay, out=dx, accumulate=accumulate, ws=ws)
        torch.cuda.synchronize()
        check()
        assert max_rel_err(to_host(dx, lay), want + old if accumulate else want) <= tol


@pytest.mark.parametrize("dtype,tile", TILES)
def test_every_tile_grouped(dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, cg, kg, G, H, W = 2, 16, 24, 3, 9, 13
    x = on_grid(gen.normal(950, 0, (N, G * cg, H, W)), dtype)
    w = on_grid(gen.he_normal(950, 1, (G * kg, cg, 3, 3)), dtype)
    dy = on_grid(gen.normal(950, 2, (N, G * kg, H, W)), dtype)
    gx, gw, gdy = (to_gpu(a, dtype, B.NSK_NHWC) for a in (x, w, dy))
    y = B.conv2d_grouped_fwd(gx, gw, G, 1, 1)
    dx = B.conv2d_grouped_dgrad(gdy, gw, x.shape, G, 1, 1)
    for g in range(G):
        c, k = slice(g * cg, (g + 1) * cg), slice(g * kg, (g + 1) * kg)
        assert max_rel_err(to_host(y, B.NSK_NHWC)[:, k], oracle.conv2d_fwd(x[:, c], w[k], 1, 1, 1)) <= TOL[dtype]
        assert max_rel_err(to_host(dx, B.NSK_NHWC)[:, c], oracle.conv2d_dgrad(dy[:, k], w[k], x[:, c].shape, 1, 1, 1)) <= TOL[dtype]


@pytest.mark.parametrize("C,R", [(8, 1), (24, 3), (72, 1)])     # one, four and two k-tiles
def test_128_by_64_tile_with_two_blocks_on_a_cu(C, R, nsk_env):
    """More than 256 blocks of it (132 x 2 here): three stages instead of four."""
    nsk_env("NSK_IGEMM_TILE", "4")
    N, H, W, K, lay, ws = 1, 129, 130, 72, B.NSK_NHWC, B.Workspace()
    print(f"pipelined kernel, 128 x 64 tile, 264 blocks, C={C} R={R}", flush=True)
    x = on_grid(gen.normal(955, 0, (N, C, H, W)), "bf16")
    w = on_grid(gen.he_normal(955, 1, (K, C, R, R)), "bf16")
    gx, gw = to_gpu(x, "bf16", lay), to_gpu(w, "bf16", lay)
    y, check = guarded((N, H, W, K), torch.bfloat16)
    B.conv2d_fwd(gx, gw, 1, R // 2, 1, lay, out=y, ws=ws)
    torch.cuda.synchronize()
    check()
    assert max_rel_err(to_host(y, lay), oracle.conv2d_fwd(x, w, 1, R // 2, 1)) <= TOL["bf16"]


@pytest.mark.parametrize("N,C,H,K,R,stride", [(24, 128, 28, 512, 1, 1), (48, 256, 28, 256, 1, 1), (80, 512, 28, 64, 1, 1), (6, 192, 14, 192, 3, 1),
                                              (55, 448, 37, 16, 1, 1)])
def test_statistics_do_not_change_the_output(N, C, H, K, R, stride):
    """Taking them may change the tile, never the order of a sum."""
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((N, H, H, C), generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn((K, R, R, C), generator=g, device="cuda")).bfloat16()
    ws = B.Workspace()
    y = B.conv2d_fwd(x, w, stride, R // 2, ws=ws)
    ys, stats = B.conv2d_fwd_stats(x, w, stride, R // 2, ws=ws)
    assert torch.equal(y, ys)
    want = y.double().sum((0, 1, 2))
    scale = (y.double() ** 2).sum((0, 1, 2)).mul(y.numel() / K).sqrt()
    assert float(((stats[0].double().sum(0) - want).abs() / scale).max()) <= 1e-6      # as the other statistics tests


# N, C, H, W, K, R, S, stride, pad: strided backward-data passes whose classes share a launch
CLASSES = [
    (2, 16, 9, 12, 24, 3, 3, 2, 1),            # four classes of 1, 2, 2, 4 taps, odd height
    (3, 40, 10, 8, 32, 1, 1, 2, 0),            # one class with a tap, three that are only zeros
    (2, 16, 7, 7, 16, 2, 2, 2, 0),             # cells past the last window belong to no tap
    (1, 8, 11, 9, 24, 5, 3, (2, 1), (2, 1)),   # two classes
]


@pytest.mark.parametrize("dtype,tile", [("f32", 0), ("bf16", 0)] + TILES)
@pytest.mark.parametrize("i", range(len(CLASSES)))
def test_strided_backward_data_in_one_launch(i, dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    N, C, H, W, K, R, S, st, pd = CLASSES[i]
    w = on_grid(gen.he_normal(970 + i, 1, (K, C, R, S)), dtype)
    P, Q = oracle.conv2d_out_dims((N, C, H, W), w.shape, st, pd, 1)
    dy = on_grid(gen.normal(970 + i, 2, (N, K, P, Q)), dtype)
    old = on_grid(gen.normal(970 + i, 3, (N, C, H, W)), dtype)
    want = oracle.conv2d_dgrad(dy, w, (N, C, H, W), st, pd, 1)
    for lay in (B.NSK_NHWC, B.NSK_NCHW):
        gw, gdy, ws = to_gpu(w, dtype, lay), to_gpu(dy, dtype, lay), B.Workspace()
        gold = to_gpu(old, dtype, lay)
        for accumulate in (False, True):
            dx, check = guarded(gold.shape, torch_dtype(dtype))
            if accumulate:
                dx.copy_(gold)
            B.conv2d_dgrad(gdy, gw, (N, C, H, W), st, pd, 1, lay, out=dx, accumulate=accumulate, ws=ws)
            torch.cuda.synchronize()
            check()
            got = to_host(dx, lay)
            assert max_rel_err(got, want + old if accumulate else want) <= TOL[dtype]
            if not accumulate:
                assert np.all(got[want == 0.0] == 0.0)


@pytest.mark.parametrize("accumulate", [False, True])
def test_small_f32_64_to_64_layer(accumulate):
    x, dy = (on_grid(gen.normal(975, t, (3, 64, 16, 32)), "f32") for t in (0, 2))
    w = on_grid(gen.he_normal(975, 1, (64, 64, 3, 3)), "f32")
    gx, gw, gdy = (to_gpu(a, "f32", B.NSK_NHWC) for a in (x, w, dy))
    assert max_rel_err(to_host(B.conv2d_fwd(gx, gw, 1, 1), B.NSK_NHWC), oracle.conv2d_fwd(x, w, 1, 1, 1)) <= TOL["f32"]
    want = oracle.conv2d_dgrad(dy, w, x.shape, 1, 1, 1) + (x if accumulate else 0)
    dx = B.conv2d_dgrad(gdy, gw, x.shape, 1, 1, out=gx.clone(), accumulate=accumulate)
    assert max_rel_err(to_host(dx, B.NSK_NHWC), want) <= TOL["f32"]


# Statistics of every kernel that leaves them: sums over lanes that hold 8 (fp32 4) channels of 64, 32 or 16, and the two-stage tile for short
# reductions, forced (7) and by its rule (513 blocks of 256 x 128 and more).  Float sums of n stored values: sqrt(n) roundings of the largest.
@pytest.mark.parametrize("tile,dtype,N,C,H,K,R,stride", [
    (7, "bf16", 3, 40, 13, 136, 1, 1), (7, "bf16", 2, 64, 11, 72, 3, 1), (7, "bf16", 2, 16, 9, 264, 3, 2), (0, "bf16", 43, 64, 56, 136, 1, 1),
    (0, "bf16", 9, 16, 33, 16, 3, 1), (0, "bf16", 9, 32, 33, 32, 3, 1), (0, "bf16", 40, 64, 48, 256, 1, 1), (0, "bf16", 5, 64, 56, 64, 3, 1),
    (0, "bf16", 4, 128, 28, 128, 3, 1), (0, "bf16", 6, 64, 56, 64, 3, 2), (0, "bf16", 3, 3, 64, 64, 7, 2), (0, "f32", 4, 64, 32, 64, 3, 1)])
def test_statistics_of_every_kernel(tile, dtype, N, C, H, K, R, stride, nsk_env):
    if tile:
        nsk_env("NSK_IGEMM_TILE", str(tile))
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((N, H, H, C), generator=g, device="cuda").to(torch_dtype(dtype))
    w = (torch.randn((K, R, R, C), generator=g, device="cuda") * (2.0 / (C * R * R)) ** 0.5).to(torch_dtype(dtype))
    y, stats = B.conv2d_fwd_stats(x, w, stride, R // 2, 1, B.NSK_NHWC)
    plain = B.conv2d_fwd(x, w, stride, R // 2)
    want = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2).cpu().double(), w.permute(0, 3, 1, 2).cpu().double(), stride=stride, padding=R // 2)
    got = y.permute(0, 3, 1, 2).cpu().double()
    assert max_rel_err(got.numpy(), want.numpy()) <= TOL[dtype]
    assert torch.equal(y, plain)
    sums, n = stats.double().sum(1).cpu(), got[:, 0].numel()
    bar = 6e-8 * n ** 0.5
    assert float((sums[0] - got.sum((0, 2, 3))).abs().max()) <= bar * float((got ** 2).sum((0, 2, 3)).max()) ** 0.5 * n ** 0.5
    assert float(((sums[1] - (got ** 2).sum((0, 2, 3))) / (got ** 2).sum((0, 2, 3))).abs().max()) <= bar


# Tiles of 256 positions of the padded coarse image (H / 2 + 3 rows of W / 2 + 3), a quarter of a thousand blocks: more than 1024 tiles give each block a run
# of five and take its ring of 864 positions around more than once.  Narrowest, ordinary and widest rows, an image that ends inside a tile.
@pytest.mark.parametrize("N,H,W", [(340, 400, 2), (64, 130, 130), (20, 226, 226), (3, 46, 30)])
def test_image_stem_backward_data_over_runs_of_tiles(N, H, W):
    print(f"stem backward-data {N} {H} {W}", flush=True)
    g = torch.Generator().manual_seed(N)
    w, dy = torch.randn(64, 3, 7, 7, generator=g).mul(0.1).bfloat16(), torch.randn(N, 64, H // 2, W // 2, generator=g).bfloat16()
    nhwc = lambda t: t.permute(0, 2, 3, 1).contiguous().cuda()
    got, check = guarded((N, H, W, 3), torch.bfloat16)
    B.conv2d_dgrad(nhwc(dy), nhwc(w), (N, 3, H, W), 2, 3, out=got)
    torch.cuda.synchronize()
    check()
    want = torch.nn.grad.conv2d_input((N, 3, H, W), w.double(), dy.double(), stride=2, padding=3)
    err = (got.permute(0, 3, 1, 2).cpu().double() - want).abs()
    # rounding to bf16: 2^-8 of the value; the sum of at most 1024 products in fp32: far below 2^-12 of its size, one unit of 6.4
    assert bool((err <= want.abs() * 2.0 ** -8 + 2.0 ** -10).all())


# The copies around a stem read and write two neighbouring pixels of an NHWC row as words, and NCHW images element by element.  Values
# are only moved, so both give the same bits.
@pytest.mark.parametrize("C,R", [(1, 3), (2, 5), (3, 7), (4, 3)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_image_stem_copies(dtype, C, R):
    x, old = (on_grid(gen.normal(980 + C, k, (3, C, 18, 26)), dtype) for k in range(2))
    w = on_grid(gen.he_normal(980 + C, 2, (64, C, R, R)), dtype)
    y, dx = {}, {}
    for lay in (B.NSK_NHWC, B.NSK_NCHW):
        gw = to_gpu(w, dtype, lay)
        gy = B.conv2d_fwd(to_gpu(x, dtype, lay), gw, 2, R // 2, 1, lay)
        y[lay] = to_host(gy, lay)
        for accumulate in (False, True):
            got = B.conv2d_dgrad(gy, gw, x.shape, 2, R // 2, 1, lay, out=to_gpu(old, dtype, lay), accumulate=accumulate)
            dx[lay, accumulate] = to_host(got, lay)
    assert max_rel_err(y[B.NSK_NHWC], oracle.conv2d_fwd(x, w, 2, R // 2, 1)) <= TOL[dtype]
    assert np.array_equal(y[B.NSK_NHWC], y[B.NSK_NCHW])
    for accumulate in (False, True):
        want = oracle.conv2d_dgrad(y[B.NSK_NHWC], w, x.shape, 2, R // 2, 1) + (old if accumulate else 0)
        assert max_rel_err(dx[B.NSK_NHWC, accumulate], want) <= TOL[dtype]
        assert np.array_equal(dx[B.NSK_NHWC, accumulate], dx[B.NSK_NCHW, accumulate])


# A row of sums a wavefront row, or the sum of four and what rounding it cut off: 32 pixels of 2^19 in the first wavefront row and a 1 in a later one
# add up to 2^24 + 1 (squares 2^43 + 1), which no single float holds.
@pytest.mark.parametrize("dtype,tile", TILES)
def test_statistics_round_no_block(dtype, tile, nsk_env):
    nsk_env("NSK_IGEMM_TILE", str(tile))
    x, w = torch.zeros(1, 16, 16, 8, device="cuda"), torch.zeros(8, 1, 1, 8, device="cuda")
    x.view(256, 8)[:32, 0], x.view(256, 8)[64, 0], w[:, 0, 0, 0] = 2.0 ** 19, 1.0, 1.0
    y, stats = B.conv2d_fwd_stats(x.to(torch_dtype(dtype)), w.to(torch_dtype(dtype)), 1, 0)
    assert torch.equal(stats[0].double().sum(0).cpu(), torch.full((8,), 2.0 ** 24 + 1, dtype=torch.float64))
    assert torch.equal(stats[1].double().sum(0).cpu(), torch.full((8,), 2.0 ** 43 + 1, dtype=torch.float64))


# The order of those sums, on one block of 32 pixels: a lane adds up every eighth, then neighbours, pairs and halves come together.
def test_order_of_the_statistics(nsk_env):
    nsk_env("NSK_IGEMM_TILE", "6")
    x, w = gen.normal(985, 0, (1, 8, 4, 8)), gen.he_normal(985, 1, (32, 8, 1, 1))
    y, stats = B.conv2d_fwd_stats(to_gpu(x, "f32", B.NSK_NHWC), to_gpu(w, "f32", B.NSK_NHWC), 1, 0)
    p = y.reshape(4, 8, 32).cpu().numpy()
    s = ((p[0] + p[1]) + p[2]) + p[3]
    s = s[0::2] + s[1::2]
    s = s[0::2] + s[1::2]
    assert np.array_equal((s[0] + s[1]).astype(np.float32), stats[0, 0].cpu().numpy())
