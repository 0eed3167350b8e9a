"""Batch-norm of the channel counts whose vectors divide a block (powers of two), NHWC: sums in chunks of channels, finished by the apply
pass up to 16 MB a tensor and by a launch of their own above, thousands of rows of statistics folded first.  Both directions
against torch in 64 bits, at the lines between the routes and at the ends of their ranges."""
import pytest
import torch

from paper_2409_11600_amd import binding as B
from parity import torch_dtype

pytestmark = pytest.mark.gpu

SHAPES = [  # N, H, W, C
    (1, 1, 1, 8),          # one row, less than a block's
    (2, 7, 7, 8), (3, 5, 5, 16), (2, 9, 9, 64), (1, 13, 11, 128), (2, 6, 7, 256), (3, 5, 4, 1024),
    (64, 46, 45, 64),      # bf16: 16.2 MiB, fp32: 32.3 MiB: a launch for the finish (fp32: small blocks for the sums of a masked pass)
    (64, 45, 45, 64),      # bf16: 15.8 MiB: finished by the apply pass
    (32, 33, 31, 256),     # two chunks of 128 channels, rows that no block's share divides
]


def _bound_sums(got, want, terms):
    # float chains of at most 100 terms, the rest in 64 bits, one rounding to float: 100 * 2^-24 of the sum of magnitudes
    assert ((got.double() - want).abs() <= 6e-6 * terms + 1e-30).all()


def _bound_values(got, want, dtype, scale):
    # one rounding to the stored type; fp32 coefficients times values, terms of size `scale`, a handful of roundings
    eps = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -22
    assert ((got.double() - want).abs() <= eps * want.abs() + 2.0 ** -21 * scale).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C", SHAPES)
def test_both_directions(N, H, W, C, dtype):
    print(f"bn chunks {N}x{H}x{W}x{C} {dtype}", flush=True)
    dt = torch_dtype(dtype)
    g = torch.Generator(device="cuda:0").manual_seed(31 * C + N)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    x, res, dout = (1.0 + r(N, H, W, C)).to(dt), r(N, H, W, C).to(dt), r(N, H, W, C).to(dt)
    gamma, beta = 1 + 0.2 * r(C), 0.2 * r(C)
    M = N * H * W
    x64, X = x.double(), x.double().reshape(M, C)
    mean, var = X.mean(0), X.var(0, unbiased=False)
    invstd = torch.rsqrt(var + 1e-5)
    z = (x64 - mean) * (invstd * gamma.double()) + beta.double() + res.double()
    scale = float((((x64.abs() + mean.abs()) * (invstd * gamma.double())) + beta.double().abs() + res.double().abs()).max())
    mask = torch.zeros(B.bn_mask_bytes(x), dtype=torch.uint8, device="cuda:0")
    rows = [None, 1, 7] + ([3136] if M >= 3136 else [])
    for n in rows:                  # its own statistics, or rows that a convolution left
        stats = None
        if n is not None:
            stats = torch.zeros((2, n, C), dtype=torch.float32, device="cuda:0")
            for k in range(n):
                share = X[k * M // n:(k + 1) * M // n]
                stats[0, k], stats[1, k] = share.sum(0).float(), (share * share).sum(0).float()
        run_m, run_v = torch.zeros(C, device="cuda:0"), torch.ones(C, device="cuda:0")
        out, m, i = B.bn_relu_add_fwd(x, gamma, beta, res, relu_mask=mask, stats=stats, running_mean=run_m, running_var=run_v)
        torch.cuda.synchronize()
        assert ((m.double() - mean).abs() <= 6e-6 * X.abs().mean(0)).all()
        # E[x^2] - E[x]^2 of sums in fp32 loses up to 2^-24 * E[x^2] (not around a shift) of the variance
        slack = 1.2e-7 * (X * X).mean(0) / (var + 1e-5) * (16 if n else 100)
        assert ((i.double() - invstd).abs() <= invstd * (6e-6 + slack)).all()
        _bound_values(out, torch.relu((x64 - m.double()) * (i.double() * gamma.double()) + beta.double() + res.double()), dtype, scale)
        assert torch.allclose(run_m.double(), 0.1 * mean, rtol=1e-4, atol=1e-6)
        bits = (out.reshape(-1, 16 // out.element_size()) > 0).long()
        assert torch.equal(mask.long(), (bits << torch.arange(bits.shape[1], device="cuda:0")).sum(1))
    dz = torch.where(out.double() > 0, dout.double(), torch.zeros((), dtype=torch.float64, device="cuda:0"))
    xhat = (x64 - m.double()) * i.double()
    sums = dz.reshape(M, C).sum(0), (dz * xhat).reshape(M, C).sum(0)
    terms = dz.abs().reshape(M, C).sum(0), (dz * xhat).abs().reshape(M, C).sum(0)
    dx64 = (gamma.double() * i.double()) * (dz - sums[0] / M - xhat * (sums[1] / M))
    for handed in (mask, None):
        for relu in (True, False) if handed is None else (True,):
            dx, dr, dg, db = B.bn_relu_add_bwd(x, out, dout, gamma, m, i, relu=relu, want_dresidual=True, relu_mask=handed)
            torch.cuda.synchronize()
            if relu:
                _bound_sums(db, sums[0], terms[0])
                _bound_sums(dg, sums[1], terms[1])
                _bound_values(dx, dx64, dtype, float(((dz.abs() + (sums[0] / M).abs() + (xhat.abs() + 1) * (sums[1] / M).abs()) * (gamma * i).abs().double()).max()))
                assert torch.equal(dr.double(), dz)
            else:
                _bound_sums(db, dout.double().reshape(M, C).sum(0), dout.double().abs().reshape(M, C).sum(0))
                assert torch.equal(dr, dout)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_bad_value_stays_in_its_channel(value):
    """Infinity or NaN in one element: its channel's statistics and gradients are bad, those of the others what they were."""
    x = torch.randn(4, 9, 9, 128, device="cuda:0").bfloat16()
    dout, gamma, beta = torch.randn_like(x), torch.ones(128, device="cuda:0"), torch.zeros(128, device="cuda:0")
    keep = torch.arange(128, device="cuda:0") != 70
    out, m, i = B.bn_relu_add_fwd(x, gamma, beta)
    clean = [t.clone() for t in (out, m, i, *B.bn_relu_add_bwd(x, out, dout, gamma, m, i))if t is not None]
    x[1, 2, 3, 70] = value
    out, m, i = B.bn_relu_add_fwd(x, gamma, beta)
    bad = [t for t in (out, m, i, *B.bn_relu_add_bwd(x, out, dout, gamma, m, i)) if t is not None]
    torch.cuda.synchronize()
    assert not torch.isfinite(m[70])
    assert all(torch.equal(a[..., keep], b[..., keep]) for a, b in zip(clean, bad))


@pytest.mark.parametrize("shape", [(40, 28, 28, 64), (64, 56, 56, 64), (120, 28, 28, 64)])     # own statistics by each route: three launches, 25, 12 MB
def test_in_place(shape):
    """out = x forward, dx = dout backward: what separate buffers give (the first row, which the statistics are shifted by, included)."""
    x = (5 + torch.randn(shape, device="cuda:0")).bfloat16()
    dout, gamma, beta = torch.randn_like(x), 1 + 0.1 * torch.randn(64, device="cuda:0"), torch.randn(64, device="cuda:0")
    for _ in range(3):
        out, m, i = B.bn_relu_add_fwd(x, gamma, beta)
        dx, _, dg, db = B.bn_relu_add_bwd(x, out, dout, gamma, m, i)
        y, g = x.clone(), dout.clone()
        out2, m2, i2 = B.bn_relu_add_fwd(y, gamma, beta, out=y)
        dx2, _, dg2, db2 = B.bn_relu_add_bwd(x, out, g, gamma, m, i, dx=g)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in ((out, out2), (m, m2), (i, i2), (dx, dx2), (dg, dg2), (db, db2)))


def test_float_chains_of_a_large_tensor():
    """Values v = 1 + 2^-10 behind a first row of zeros: v and v*v add up without an error in fp32 chains of 16 terms, not of 32 (v*v has 20
    bits behind the point).  The variance is v*v / M (1 - 1/M), 5e5 times smaller than the sums it comes from: with chains of at
    most 16 only the block with the first row rounds (2^-24 of 2048 / M of the sum: 1.2e-4 of the variance)."""
    N, H, W, C = 128, 64, 64, 64
    M, v = N * H * W, 1 + 2.0 ** -10
    x = torch.full((N, H, W, C), v, device="cuda:0")
    x[0, 0, 0] = 0
    _, m, i = B.bn_relu_add_fwd(x, torch.ones(C, device="cuda:0"), torch.zeros(C, device="cuda:0"), eps=0.0)
    torch.cuda.synchronize()
    assert torch.allclose(m.double(), torch.full_like(m, 1.0).double() * v * (1 - 1 / M), rtol=1e-6)
    want = (v * v / M * (1 - 1 / M)) ** -0.5
    assert ((i.double() - want).abs() <= 1e-3 * want).all()


@pytest.mark.parametrize("M,C,dtype,rows", [
    (3200, 64, "bf16", (200, 201, 1024, 1025)),        # 100 KB of sums a chunk; the line of the fold
    (12900, 16, "bf16", (1600, 1601)),                 # 200 KB up to 32 channels
    (3200, 256, "f32", (100, 101)),                    # two chunks of 128 channels
    (2100, 512, "bf16", (220, 221, 512, 513)),
    (1100, 1024, "f32", (512, 513)),
    (4096, 512, "bf16", (None,)), (4095, 512, "bf16", (None,)),          # 4 MB: own sums in chunks, or over whole rows
    (1024, 1024, "bf16", (None,)), (20480, 128, "f32", (None,)), (20479, 128, "f32", (None,)),      # 10 MB
    (131072, 64, "bf16", (None,)), (131071, 64, "bf16", (None,)),                                   # 16 MB: its finish
])
def test_forward_routes(M, C, dtype, rows):
    """Both sides of the lines between the forward routes: statistics of a convolution that the apply pass reads, that a launch between
    finishes, that are folded first; own statistics by either kernel.  Against torch in 64 bits."""
    dt = torch_dtype(dtype)
    g = torch.Generator(device="cuda:0").manual_seed(M + C)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    x, gamma, beta = (0.3 + r(M, 1, 1, C)).to(dt), 1 + 0.2 * r(C), 0.2 * r(C)
    X = x.double().reshape(M, C)
    mean, var = X.mean(0), X.var(0, unbiased=False)
    invstd = torch.rsqrt(var + 1e-5)
    for n in rows:
        print(f"bn forward routes {M}x{C} {dtype} rows {n}", flush=True)
        stats = None
        if n is not None:
            at = torch.arange(M, device="cuda:0") * n // M                  # disjoint shares of the rows
            stats = torch.stack([torch.zeros(n, C, dtype=torch.float64, device="cuda:0").index_add_(0, at, v) for v in (X, X * X)]).float()
        out, m, i = B.bn_relu_add_fwd(x, gamma, beta, stats=stats)
        torch.cuda.synchronize()
        # rows rounded to float (exact sums otherwise), or float chains of at most 100 terms; then E[x^2] - E[x]^2 in 64 bits
        assert ((m.double() - mean).abs() <= 6e-6 * X.abs().mean(0)).all()
        assert ((i.double() - invstd).abs() <= 1.4e-5 * invstd).all()
        want = torch.relu((X - m.double()) * (i.double() * gamma.double()) + beta.double()).view_as(out)
        scale = float(((X.abs() + m.double().abs()) * (i * gamma).abs().double() + beta.abs().double()).max())
        _bound_values(out, want, dtype, scale)
