"""Backward-weight of 3x3 layers with 16 channels: whole images and strips, fewer images than CUs, ragged last strips and runs, more strips than
blocks, one pixel under the line to the pipelined kernel, accumulation, against torch in 64 bits on the device."""
import ctypes

import pytest
import torch

from paper_2409_11600_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W", [(256, 32, 32), (300, 16, 16), (21, 56, 56), (1, 256, 256), (1, 255, 257), (70, 31, 33), (530, 19, 15), (1100, 16, 16),
                                   (30, 2, 1100), (40, 61, 29), (1, 700, 100)])
def test_backward_weight(N, H, W, C=16, K=16):
    print(f"narrow backward-weight {N}x{H}x{W} {C}->{K}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N + H + C)
    r = lambda *s: torch.randn(s, generator=g, device="cuda:0")
    x, dy, old = r(N, H, W, C).bfloat16(), r(N, H, W, K).bfloat16(), r(K, 3, 3, C)
    dw = B.conv2d_wgrad(x, dy, (K, C, 3, 3), 1, 1)
    acc = B.conv2d_wgrad(x, dy, (K, C, 3, 3), 1, 1, out=old.clone(), accumulate=True)
    torch.cuda.synchronize()
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    D = dy.double().reshape(-1, K).t()
    shifted = lambda X, a, b: X[:, a:a + H, b:b + W].reshape(-1, C)
    want = torch.stack([torch.stack([D @ shifted(xp, a, b) for b in range(3)], 1) for a in range(3)], 1)
    size = torch.stack([torch.stack([D.abs() @ shifted(xp.abs(), a, b) for b in range(3)], 1) for a in range(3)], 1)
    # exact products; fp32 chains of 32 products, of strips and of blocks
    assert ((dw.double() - want).abs() <= 2e-5 * size).all()
    assert ((acc.double() - want - old.double()).abs() <= 2e-5 * (size + old.double().abs())).all()
    assert torch.equal(dw, B.conv2d_wgrad(x, dy, (K, C, 3, 3), 1, 1))


def test_the_largest_operands():
    """67.0 M pixels, 2.1 GB an operand: offsets up to 2^31 bytes, one image more is refused.  x is zero but for the last 23 images, which
    are the ones that the reference adds up."""
    N, H, W, C, first = 1023, 256, 256, 16, 1000
    print(f"narrow backward-weight {N}x{H}x{W}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N)
    x, dy = torch.zeros((N, H, W, C), device="cuda:0", dtype=torch.bfloat16), torch.ones((N, H, W, C), device="cuda:0", dtype=torch.bfloat16)
    for t in (x, dy):
        t[first:] = torch.randn((N - first, H, W, C), generator=g, device="cuda:0")
    dw = B.conv2d_wgrad(x, dy, (C, C, 3, 3), 1, 1)
    torch.cuda.synchronize()
    xp = torch.nn.functional.pad(x[first:].double(), (0, 0, 1, 1, 1, 1))
    D = dy[first:].double().reshape(-1, W, C).transpose(1, 2).contiguous()          # a product per image row
    shifted = [[xp[:, r:r + H, s:s + W].reshape(-1, W, C).contiguous() for s in range(3)] for r in range(3)]
    stack = lambda A, f: torch.stack([torch.stack([torch.bmm(A, f(X)).sum(0) for X in row], 1) for row in shifted], 1)
    want, size = stack(D, lambda X: X), stack(D.abs(), torch.abs)
    assert ((dw.double() - want).abs() <= 2e-5 * size).all()
    more = B.conv_desc((N + 1, C, H, W), (C, 3, 3), 1, 1, 1, B.NSK_BF16, B.NSK_NHWC)
    status = B.lib().nsk_conv2d_wgrad(ctypes.byref(more), B._ptr(x), B._ptr(dy), B._ptr(dw), 0, None, 0, B._stream())
    assert status == B.NSK_ERR_UNSUPPORTED
