"""Backward-weight of 3x3 layers with 16 channels: whole images and strips, fewer images than CUs, ragged last strips and runs, more strips than
blocks, one pixel under the line to the pipelined kernel, accumulation, against torch in 64 bits on the device."""
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
