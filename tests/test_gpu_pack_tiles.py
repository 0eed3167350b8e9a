"""The filter packing of backward-data by tiles (both channel counts of at least 32 and whole vectors, large filters) and by the gather
(small ones): channel counts that no tile divides, every residue class of a strided filter, grouped filters, against torch in 64 bits
on the CPU."""
import pytest
import torch

from paper_2409_11600_amd import binding as B
from parity import TOL, max_rel_err, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,K,R,stride,groups", [(32, 32, 1, 1, 1), (40, 72, 3, 1, 1), (136, 40, 3, 2, 1), (64, 200, 2, 2, 1), (80, 64, 3, 1, 2), (136, 144, 3, 1, 1), (520, 408, 2, 2, 1), (136, 120, 3, 1, 2),
                                                 (72, 32, 1, 2, 1), (24, 64, 3, 1, 1)])
def test_backward_data(C, K, R, stride, groups, dtype):
    print(f"pack tiles {C}->{K} {R}x{R} stride {stride} groups {groups} {dtype}", flush=True)
    dt, pad = torch_dtype(dtype), R // 2
    g = torch.Generator().manual_seed(C * K)
    w = torch.randn((K * groups, R, R, C), generator=g).to(dt)
    x_shape = (2, C * groups, 9, 8)
    P, Q = ((n + 2 * pad - R) // stride + 1 for n in x_shape[2:])
    dy = torch.randn((2, P, Q, K * groups), generator=g).to(dt)
    want = torch.nn.grad.conv2d_input(x_shape, w.double().permute(0, 3, 1, 2).contiguous(), dy.double().permute(0, 3, 1, 2).contiguous(),
                                      stride=stride, padding=pad, groups=groups).permute(0, 2, 3, 1)
    if groups == 1:
        dx = B.conv2d_dgrad(dy.cuda(), w.cuda(), x_shape, stride, pad)
    else:
        dx = B.conv2d_grouped_dgrad(dy.cuda(), w.cuda(), x_shape, groups, stride, pad)
    torch.cuda.synchronize()
    assert max_rel_err(dx.double().cpu().numpy(), want.numpy()) <= TOL[dtype]
