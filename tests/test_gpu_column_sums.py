"""The reductions of a training step's tail where they can go wrong: bias gradients on both sides of the row count from which a
block has 16 columns, ragged columns; sums of squares with remainders, from one element to more than the partial sums' blocks
take in one round."""
import numpy as np
import pytest
import torch

from paper_2409_11600_amd import binding as B
from parity import guarded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,K", [(1, 7), (63, 64), (1023, 40), (1024, 40), (1024, 1), (1500, 17), (3001, 130)])
def test_bias_gradient(N, K, dtype):
    print(f"bias gradient N={N} K={K} {dtype}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(N + K)
    x, dy = (torch.randn((N, c), generator=g, device="cuda:0").to(dtype) for c in (8, K))
    old = torch.randn(K, generator=g, device="cuda:0")
    want = dy.double().sum(0)
    # float sums: a chain of at most N/16 + 16 + N/1024 roundings of partial sums below sum |dy|
    bar = (N / 16 + 32) * 2.0 ** -24 * dy.double().abs().sum(0)
    for accumulate in (False, True):
        db, ok = guarded((K,), torch.float32)
        dw = torch.zeros((K, 8), device="cuda:0")
        if accumulate:
            db.copy_(old)
        B.linear_wgrad(x, dy, dw=dw, db=db, accumulate=accumulate)
        torch.cuda.synchronize()
        ok()
        assert bool(((db.double() - want - (old.double() if accumulate else 0)).abs() <= bar + 2.0 ** -23 * old.abs()).all())


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1027, 4099, 100001, 262144 * 4 + 5, 262144 * 17 + 2])
def test_sum_of_squares(n):
    print(f"sum of squares n={n}", flush=True)
    g = torch.randn(n + 8, generator=torch.Generator(device="cuda:0").manual_seed(n), device="cuda:0")
    g[n:] = float("nan")                     # (what lies behind is not read into the sum)
    part, total = torch.empty(256, device="cuda:0"), torch.full((1,), 3.0, device="cuda:0")
    B._check(B.lib().nsk_sumsq_accumulate(n, B._ptr(g), B._ptr(part), B._ptr(total), B._stream()), "nsk_sumsq_accumulate")
    want = 3.0 + float((g[:n].double() ** 2).sum())
    assert abs(float(total) - want) <= 4 * 2.0 ** -24 * want     # squares, partial sums and the result rounded to float once each
