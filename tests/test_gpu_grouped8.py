"""Grouped bf16 3x3 layers with eight channels per group: the kernels on strips of rows, at the sizes where they can go wrong
(one pixel, one row, strips that do not divide the image, chunks of 64 channels that are not full, widths up to the last
that fits and one past it), against the oracle group by group; infinities stay with the pixels that touch them."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
import oracle
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, to_gpu, to_host, torch_dtype

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2, 1, 1), (2, 8, 1, 7), (3, 9, 5, 1), (2, 12, 15, 28), (1, 3, 31, 17), (2, 2, 9, 56), (1, 8, 3, 148), (1, 2, 3, 159), (1, 2, 4, 170)]   # N, groups, H, W


@pytest.mark.parametrize("direct", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_groups_of_eight(shape, direct, nsk_env):
    if direct:
        nsk_env("NSK_NO_GROUPED8", "1")
    N, G, H, W = shape
    print(f"groups of eight, N, groups, H, W = {shape} direct={direct}", flush=True)
    C, lay, ws = 8 * G, B.NSK_NHWC, B.Workspace()
    x, dy, old = (on_grid(gen.normal(1200, t, (N, C, H, W)), "bf16") for t in (0, 1, 2))
    w = on_grid(gen.he_normal(1200, 3, (C, 8, 3, 3)), "bf16")
    gx, gdy, gw = (to_gpu(a, "bf16", lay) for a in (x, dy, w))
    y, y_ok = guarded(gx.shape, torch.bfloat16)
    B.conv2d_grouped_fwd(gx, gw, G, 1, 1, out=y, ws=ws)
    dx, dx_ok = guarded(gx.shape, torch.bfloat16)
    B.conv2d_grouped_dgrad(gdy, gw, x.shape, G, 1, 1, out=dx, ws=ws)
    dxa = to_gpu(old, "bf16", lay)
    B.conv2d_grouped_dgrad(gdy, gw, x.shape, G, 1, 1, out=dxa, accumulate=True, ws=ws)
    dw, dw_ok = guarded((C, 3, 3, 8), torch.float32)
    B.conv2d_grouped_wgrad(gx, gdy, (C, 8, 3, 3), G, 1, 1, out=dw, ws=ws)
    torch.cuda.synchronize()
    for ok in (y_ok, dx_ok, dw_ok):
        ok()
    y, dx, dxa, dw = (to_host(t, lay) for t in (y, dx, dxa, dw))
    for g in range(G):
        c = slice(8 * g, 8 * g + 8)
        want = oracle.conv2d_dgrad(dy[:, c], w[c], x[:, c].shape, 1, 1, 1)
        assert max_rel_err(y[:, c], oracle.conv2d_fwd(x[:, c], w[c], 1, 1, 1)) <= TOL["bf16"]
        assert max_rel_err(dx[:, c], want) <= TOL["bf16"]
        assert max_rel_err(dxa[:, c], want + old[:, c]) <= TOL["bf16"]
        assert max_rel_err(dw[c], oracle.conv2d_wgrad(x[:, c], dy[:, c], (8, 8, 3, 3), 1, 1, 1)) <= TOL["f32"]


def test_infinities_stay_where_they_belong():
    N, G, H, W = 1, 4, 9, 21
    x = on_grid(gen.normal(1210, 0, (N, 8 * G, H, W)), "bf16")
    w = on_grid(gen.he_normal(1210, 1, (8 * G, 8, 3, 3)), "bf16")
    dy = on_grid(gen.normal(1210, 2, x.shape), "bf16")
    x[0, 11, 4, 10] = np.inf      # group 1
    gx, gw, gdy = (to_gpu(a, "bf16", B.NSK_NHWC) for a in (x, w, dy))
    y = to_host(B.conv2d_grouped_fwd(gx, gw, G, 1, 1), B.NSK_NHWC)
    touched = np.zeros(y.shape, bool)
    touched[0, 8:16, 3:6, 9:12] = True
    assert np.array_equal(~np.isfinite(y), touched)
    dw = to_host(B.conv2d_grouped_wgrad(gx, gdy, (8 * G, 8, 3, 3), G, 1, 1), B.NSK_NHWC)
    touched = np.zeros(dw.shape, bool)
    touched[8:16, 3] = True
    assert np.array_equal(~np.isfinite(dw), touched)
