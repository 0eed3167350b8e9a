"""The short-reduction kernel around the lines between one and two blocks a CU: 3x3 filters of 16- and 32-channel outputs and 1x1 filters of 32 and
64 channels, ragged last tiles, with statistics, against torch in 64 bits on the device."""
import pytest
import torch

from paper_2409_11600_amd import binding as B

pytestmark = pytest.mark.gpu


def conv64(x, w):
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    N, H, W, _ = x.shape
    return sum(xp[:, r:r + H, s:s + W] @ w[:, r, s].double().t() for r in range(3) for s in range(3))


@pytest.mark.parametrize("N,H,W,C,K", [(128, 32, 32, 16, 16), (127, 32, 32, 16, 16), (128, 31, 33, 32, 16), (64, 32, 32, 32, 32), (63, 33, 31, 32, 32),
                                       (131, 32, 32, 16, 32), (9, 31, 30, 16, 16)])
def test_forward_backward_data_and_statistics(N, H, W, C, K):
    print(f"narrow {N}x{H}x{W} {C}->{K}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N + H)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    x, w, dy, old = r(N, H, W, C).bfloat16(), (r(K, 3, 3, C) / (9 * C) ** 0.5).bfloat16(), r(N, H, W, K).bfloat16(), r(N, H, W, C).bfloat16()
    want = conv64(x, w)
    y, stats = B.conv2d_fwd_stats(x, w, 1, 1)
    dx = B.conv2d_dgrad(dy, w, (N, C, H, W), 1, 1)
    acc = B.conv2d_dgrad(dy, w, (N, C, H, W), 1, 1, out=old.clone(), accumulate=True)
    torch.cuda.synchronize()
    # one rounding to bf16 (2^-9 of the value) and fp32 sums of 9*C products
    near = lambda a, b: ((a.double() - b).abs() <= 2.0 ** -8 * b.abs() + 1e-5).all()
    assert near(y, want)
    dx64 = conv64(dy, w.flip(1, 2).permute(3, 1, 2, 0).contiguous())
    assert near(dx, dx64) and near(acc, dx64 + old.double())
    Y = y.double().reshape(-1, K)
    # sums of the values as stored: float chains of a few hundred
    assert ((stats[0].double().sum(0) - Y.sum(0)).abs() <= 2e-5 * Y.abs().sum(0)).all()
    assert ((stats[1].double().sum(0) - (Y * Y).sum(0)).abs() <= 2e-5 * (Y * Y).sum(0)).all()


@pytest.mark.parametrize("N,H,W,C,K", [(21, 56, 56, 64, 64), (1, 257, 255, 64, 64), (1, 257, 255, 32, 128),    # one tile under and over the line
                                       (32, 56, 57, 64, 256), (43, 57, 55, 64, 192), (64, 56, 56, 32, 64), (9, 113, 111, 256, 64),
                                       (2, 181, 183, 64, 512)])                                              # 512: columns split
def test_one_tap(N, H, W, C, K):
    print(f"one tap {N}x{H}x{W} {C}->{K}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N + H)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    x, w, dy, old = r(N, H, W, C).bfloat16(), (r(K, 1, 1, C) / C ** 0.5).bfloat16(), r(N, H, W, K).bfloat16(), r(N, H, W, C).bfloat16()
    y, stats = B.conv2d_fwd_stats(x, w, 1, 0)
    plain = B.conv2d_fwd(x, w, 1, 0)
    dx = B.conv2d_dgrad(dy, w, (N, C, H, W), 1, 0)
    acc = B.conv2d_dgrad(dy, w, (N, C, H, W), 1, 0, out=old.clone(), accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(y, plain)
    w64 = w[:, 0, 0].double()
    # one rounding to bf16 and fp32 sums of C (K) products
    near = lambda a, b: ((a.double() - b).abs() <= 2.0 ** -8 * b.abs() + 1e-5).all()
    assert near(y, x.double() @ w64.t())
    dx64 = dy.double() @ w64
    assert near(dx, dx64) and near(acc, dx64 + old.double())
    Y = y.double().reshape(-1, K)
    assert ((stats[0].double().sum(0) - Y.sum(0)).abs() <= 2e-5 * Y.abs().sum(0)).all()
    assert ((stats[1].double().sum(0) - (Y * Y).sum(0)).abs() <= 2e-5 * (Y * Y).sum(0)).all()


@pytest.mark.parametrize("C,K,R,rows", [(64, 64, 1, 64), (16, 16, 3, 64), (32, 32, 3, 32)])
def test_a_block_adds_its_wavefronts_in_64_bits(C, K, R, rows):
    """A block's four wavefronts (tiles of `rows` pixels, one after the other) leave 2^24, 1, -2^24 and 0 in its row of statistics: in fp32 the
    1 would be lost, in 64 bits nothing is."""
    N, H, W = 128, 32, 32
    big = 2.0 ** 24 / rows
    x = torch.zeros(N * H * W // (4 * rows), 4, rows, C, dtype=torch.bfloat16, device="cuda:0")
    x[:, 0], x[:, 1, 5], x[:, 2] = big, 1.0, -big
    w = torch.zeros(K, R, R, C, dtype=torch.bfloat16, device="cuda:0")
    w[:, R // 2, R // 2] = torch.eye(K)
    y, stats = B.conv2d_fwd_stats(x.view(N, H, W, C), w, 1, R // 2)
    torch.cuda.synchronize()
    assert torch.equal(y.view(-1), x.view(-1))
    assert (stats[0].double().sum(0) == x.shape[0]).all()
