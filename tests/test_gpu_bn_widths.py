"""Batch-norm on channel counts whose vectors do not divide a block of the NHWC kernels: one vector, idle threads at the end of a
block, more than one chunk of 256 vectors, 8-byte vectors in bf16, tensors below the size from which the
vectors are used; thousands of rows of statistics handed in; against the oracle and against the general path (the same values as NCHW)."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, to_gpu, to_host, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("relu,res", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C", [4, 12, 24, 36, 96, 100, 344, 520, 1028, 1032, 2056, 4100])
def test_any_width(C, dtype, relu, res):
    N, H, W = (2, 7, -(-524288 // (14 * C)) + (0 if relu else 3)) if res or C > 400 else (3, 11, 13)   # from 512 k elements on; below
    print(f"batch-norm C={C} {dtype} relu={relu} residual={res}", flush=True)
    tol, s = TOL[dtype], 7000 + C
    # means of about one: a mean comes from chains of float sums of differences of size 1..4, at most 32 long here, so it is good to
    # 32 * 2^-24 * 4 = 8e-6 in absolute terms (a mean of 0.01 has no relative bar of 1e-5)
    x, r, dout = (on_grid(gen.normal(s, k, (N, C, H, W)) + (k == 0), dtype) for k in range(3))
    gamma, beta = 1 + 0.2 * gen.normal(s, 3, (C,)).astype(np.float32), 0.2 * gen.normal(s, 4, (C,)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda:0")
    want, wmean, winv = oracle.bn_relu_add_fwd(x, gamma, beta, r if res else None, 1e-5, relu)[:3]
    wmean, winv = wmean.astype(np.float32), winv.astype(np.float32)
    kept = on_grid(want, dtype)
    wdx, wdres, wdg, wdb = oracle.bn_relu_add_bwd(x, kept, dout, gamma, wmean, winv, relu, want_dresidual=res)
    for lay in (B.NSK_NHWC, B.NSK_NCHW):
        gx, gr, gd, gk, ws = *(to_gpu(a, dtype, lay) for a in (x, r, dout, kept)), B.Workspace()
        out, ok = guarded(gx.shape, torch_dtype(dtype))
        _, mean, inv = B.bn_relu_add_fwd(gx, dev(gamma), dev(beta), gr if res else None, 1e-5, relu, lay, out=out, ws=ws)
        torch.cuda.synchronize()
        ok()
        assert max_rel_err(to_host(out, lay), want) <= tol
        assert max_rel_err(mean.cpu().numpy(), wmean) <= 1e-5 and max_rel_err(inv.cpu().numpy(), winv) <= 1e-5
        dx, ok = guarded(gx.shape, torch_dtype(dtype))
        _, dres, dg, db = B.bn_relu_add_bwd(gx, gk, gd, dev(gamma), dev(wmean), dev(winv), relu, lay, dx=dx, want_dresidual=res, ws=ws)
        torch.cuda.synchronize()
        ok()
        assert max_rel_err(to_host(dx, lay), wdx) <= tol
        assert max_rel_err(dg.cpu().numpy(), wdg) <= 1e-4 and max_rel_err(db.cpu().numpy(), wdb) <= 1e-4
        if res:
            assert np.array_equal(to_host(dres, lay), wdres)      # a masked copy: exact


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,rows,lay", [(96, 3000, B.NSK_NHWC), (100, 2000, B.NSK_NHWC), (1032, 1500, B.NSK_NHWC), (64, 5000, B.NSK_NHWC),
                                        (20, 4000, B.NSK_NCHW), (96, 1100, B.NSK_NCHW)])
def test_statistics_handed_in(C, rows, lay, dtype):
    N, H, W, s = 2, 50, 54 if lay == B.NSK_NHWC else 31, 7900 + C      # (NHWC: enough elements for the vectors)
    x = on_grid(gen.normal(s, 0, (N, C, H, W)), dtype)
    gx = to_gpu(x, dtype, lay)
    # the rows add up to the tensor's sums: as many random rows as fit, the rest in the last
    part = (0.01 * gen.normal(s, 1, (2, rows, C))).astype(np.float32)
    total = np.stack([x.sum((0, 2, 3)), (x.astype(np.float64) ** 2).sum((0, 2, 3))])
    part[:, -1] = total - part[:, :-1].astype(np.float64).sum(1)
    gamma, beta = torch.ones(C, device="cuda:0"), torch.zeros(C, device="cuda:0")
    out, mean, inv = B.bn_relu_add_fwd(gx, gamma, beta, None, 1e-5, False, lay, stats=torch.from_numpy(part).to("cuda:0"))
    want, wmean, winv = oracle.bn_relu_add_fwd(x, np.ones(C), np.zeros(C), None, 1e-5, False)[:3]
    # the last row is rounded to float and up to `rows` of size 0.01 are added in float by the fold
    assert np.abs(mean.cpu().numpy() - wmean).max() <= 1e-5 and max_rel_err(inv.cpu().numpy(), winv) <= 1e-4
    assert max_rel_err(to_host(out, lay), want) <= max(TOL[dtype], 1e-4)


def test_what_was_refused_stays_refused():
    x = torch.zeros((2, 3, 5, 96), device="cuda:0")
    assert B.bn_mask_bytes(x) == 0
    z = torch.zeros(96, device="cuda:0")
    with pytest.raises(B.NskError) as e:
        B.bn_relu_bwd_act(x, torch.zeros((2, 96), device="cuda:0"), x, z, z, z)
    assert e.value.status == B.NSK_ERR_UNSUPPORTED


@pytest.mark.parametrize("lay", [B.NSK_NHWC, B.NSK_NCHW], ids=["nhwc", "nchw"])
def test_many_rows_are_added_without_long_float_chains(lay):
    """One image's sums in 4000 rows that are far larger than their total."""
    C, rows, H, W = 20, 4000, 64, 104
    g = np.random.default_rng(5)
    part = np.stack([g.standard_normal((rows, C)), np.abs(g.standard_normal((rows, C))) + 50]).astype(np.float32)
    part[0] += np.where(np.arange(rows) < rows // 2, 100, -100).astype(np.float32)[:, None]
    shape = (1, H, W, C) if lay == B.NSK_NHWC else (1, C, H, W)
    x, one, zero = torch.zeros(shape, device="cuda:0"), torch.ones(C, device="cuda:0"), torch.zeros(C, device="cuda:0")
    _, mean, _ = B.bn_relu_add_fwd(x, one, zero, None, 1e-5, False, lay, stats=torch.from_numpy(part).to("cuda:0"))
    want = part[0].astype(np.float64).sum(0) / (H * W)
    # no run of float additions is longer than 64 rows of 104 before fp64: at most 64 roundings of 6656 in 63 runs, in a random walk
    bar = 8 * np.sqrt(64 * 63) * 2.0 ** -24 * 6656 / 2 / (H * W)
    assert np.abs(mean.cpu().numpy() - want).max() <= bar + 2.0 ** -24 * np.abs(want).max()


# A thread adds up at most eight rows here, three roundings a row, and what follows is in fp64: 2.5e-8 * sqrt(24 / 2), 2.5e-8 being
# the rms of one rounding.
@pytest.mark.parametrize("dtype,N,C,H,W", [("bf16", 95, 24, 20, 17), ("bf16", 27, 24, 40, 66), ("f32", 64, 12, 28, 28), ("f32", 64, 16, 40, 42)])
def test_sums_of_few_channels_keep_their_precision(dtype, N, C, H, W):
    g = torch.Generator(device="cuda").manual_seed(3)
    x, dy = (torch.randn((N, H, W, C), generator=g, device="cuda").to(torch_dtype(dtype)) for _ in range(2))
    one, zero = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    out, mean, inv = B.bn_relu_add_fwd(x, one, zero, None, 1e-5, True)
    _, _, dg, db = B.bn_relu_add_bwd(x, out, dy, one, mean, inv, True)
    off = lambda a, w: float((a.double() - w).norm() / w.norm())
    dz = torch.where(out > 0, dy.double(), torch.zeros((), dtype=torch.float64, device="cuda"))
    assert off(db, dz.sum((0, 1, 2))) <= 9e-8
    assert off(dg, (dz * ((x.double() - mean.double()) * inv.double())).sum((0, 1, 2))) <= 9e-8
    var = ((x.double() - x.double().mean((0, 1, 2))) ** 2).mean((0, 1, 2))
    assert off(inv, torch.rsqrt(var + 1e-5)) <= 9e-8


# N, C: G = min(1024 / C, N) blocks; either side of the lines for folding (rows x C x 8 bytes of 4 MB, 16384 rows at 48 blocks)
@pytest.mark.parametrize("N,C,rows", [(24, 40, 13000), (24, 40, 13200), (32, 32, 16300), (32, 32, 16500), (48, 8, 16300), (48, 8, 16500),
                                      (64, 8, 1100), (23, 32, 17000), (3, 20, 30000)])
def test_rows_of_statistics_either_side_of_the_fold(N, C, rows):
    g, side = np.random.default_rng(N + C + rows), int(np.sqrt(rows / N)) + 1
    part = np.stack([g.standard_normal((rows, C)) + 1, np.abs(g.standard_normal((rows, C))) + 3]).astype(np.float32)
    x, one, zero = torch.zeros((N, C, side, side), device="cuda:0"), torch.ones(C, device="cuda:0"), torch.zeros(C, device="cuda:0")
    _, mean, inv = B.bn_relu_add_fwd(x, one, zero, None, 1e-5, False, B.NSK_NCHW, stats=torch.from_numpy(part).to("cuda:0"))
    n = N * side * side
    s = part.astype(np.float64).sum(1) / n
    # the rows are added in fp64; a folded row, mean and invstd are each rounded to float once
    assert max_rel_err(mean.cpu().numpy(), s[0]) <= 2.0 ** -23
    assert max_rel_err(inv.cpu().numpy(), 1 / np.sqrt(s[1] - s[0] ** 2 + 1e-5)) <= 2.0 ** -23 * (s[1] + 2 * s[0] ** 2).max() / (s[1] - s[0] ** 2).min()
