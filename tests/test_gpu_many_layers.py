"""The calls that pack filters and add up partial sums for many layers at once: bit by bit the results of each layer's own calls, for every
kind of layer that they take, more layers than one launch holds, and the layers that they refuse."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2409_11600_amd import binding as B, network
from parity import torch_dtype

pytestmark = pytest.mark.gpu

# dtype, N, C, H, K, R, stride
LAYERS = [("bf16", 16, 16, 32, 16, 3, 1), ("bf16", 8, 3, 32, 16, 3, 1), ("bf16", 16, 16, 32, 32, 3, 2), ("bf16", 16, 16, 32, 32, 1, 2), ("bf16", 16, 32, 16, 32, 3, 1),
          ("bf16", 16, 64, 8, 64, 3, 1), ("bf16", 40, 64, 24, 64, 3, 1), ("bf16", 4, 96, 9, 40, 1, 1), ("bf16", 3, 24, 7, 72, 3, 2), ("f32", 8, 16, 32, 16, 3, 1),
          ("f32", 4, 64, 16, 64, 3, 1), ("f32", 2, 20, 9, 36, 3, 2),
          ("f32", 4, 16, 14, 64, 1, 2)]      # (its tile goes by the pixels that no tap reaches, too)


def _layer(dtype, N, C, H, K, R, st, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch_dtype(dtype))
    P = (H + 2 * (R // 2) - R) // st + 1
    d = B.conv_desc((N, C, H, H), (K, R, R), st, R // 2, 1, B._dtype_code(r(1)), B.NSK_NHWC)
    return d, r(N, H, H, C), r(K, R, R, C), r(N, P, P, K)


def _items(of):
    return len(of), (B.nsk_conv_item_t * len(of))(*[(ctypes.pointer(d), s.data_ptr(), t.data_ptr()) for d, s, t in of])


def _ok(status):
    assert status == B.NSK_OK, status


@pytest.mark.parametrize("copies", [1, 7])      # 7: 91 layers, more than one launch holds
def test_many_layers_at_once(copies):
    L, ptr = B.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    layers = [_layer(*l, seed=i) for i, l in enumerate(LAYERS * copies)]
    packs, sums, want = [], [], []
    for d, x, w, dy in layers:
        fb, pb = L.nsk_conv2d_packed_filter_bytes(ctypes.byref(d)), L.nsk_conv2d_wgrad_partial_bytes(ctypes.byref(d))
        assert fb > 0 or d.C == 3 or d.K % 8 or d.C % 8      # (channel counts that are copied to whole vectors keep their own calls)
        if fb:
            packs.append((d, w, torch.full((fb,), 255, dtype=torch.uint8, device="cuda")))
        if pb:
            sums.append((d, torch.full((pb // 4,), float("nan"), device="cuda"), torch.full(w.shape, float("nan"), device="cuda")))
    assert len(packs) >= 9 * copies and len(sums) >= 9 * copies
    _ok(L.nsk_conv2d_pack_filters(*_items(packs), st))
    packed, partial = {id(d): t for d, _, t in packs}, {id(d): (p, t) for d, p, t in sums}
    for d, x, w, dy in layers:
        if id(d) in partial:
            _ok(L.nsk_conv2d_wgrad_partial(ctypes.byref(d), ptr(x), ptr(dy), ptr(partial[id(d)][0]), st))
    _ok(L.nsk_conv2d_wgrad_reduce(*_items(sums), 0, st))
    for i, (d, x, w, dy) in enumerate(layers):
        dims = (d.N, d.C, d.H, d.W)
        if id(d) in partial:
            own = B.conv2d_wgrad(x, dy, (d.K, d.C, d.R, d.S), d.stride_h, d.pad_h)
            assert torch.equal(partial[id(d)][1], own), LAYERS[i % len(LAYERS)]
        if id(d) in packed:
            for acc in (0, 1):
                got = x.clone()
                _ok(L.nsk_conv2d_dgrad_packed(ctypes.byref(d), ptr(dy), ptr(packed[id(d)]), ptr(got), acc, st))
                own = B.conv2d_dgrad(dy, w, dims, d.stride_h, d.pad_h, out=x.clone(), accumulate=bool(acc))
                assert torch.equal(got, own), (LAYERS[i % len(LAYERS)], acc)
    _ok(L.nsk_conv2d_wgrad_reduce(*_items(sums), 1, st))
    for i, (d, x, w, dy) in enumerate(layers):
        if id(d) in partial:
            own = B.conv2d_wgrad(x, dy, (d.K, d.C, d.R, d.S), d.stride_h, d.pad_h)
            assert torch.equal(partial[id(d)][1], own + own), LAYERS[i % len(LAYERS)]


def test_layers_that_keep_their_own_calls():
    L, ptr = B.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for dims, filt, stride, pad, layout in (((2, 16, 8, 8), (16, 3, 3), 1, 1, B.NSK_NCHW), ((2, 512, 8, 8), (512, 3, 3), 1, 1, B.NSK_NHWC),
                                            ((2, 16, 16, 16), (16, 5, 5), 1, 2, B.NSK_NHWC), ((2, 16, 16, 16), (16, 3, 3), 3, 1, B.NSK_NHWC),
                                            ((2, 3, 32, 32), (64, 7, 7), 2, 3, B.NSK_NHWC)):
        d = B.conv_desc(dims, filt, stride, pad, 1, B.NSK_BF16, layout)
        assert L.nsk_conv2d_packed_filter_bytes(ctypes.byref(d)) == 0
        t = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
        assert L.nsk_conv2d_pack_filters(1, (B.nsk_conv_item_t * 1)((ctypes.pointer(d), t.data_ptr(), t.data_ptr())), st) == B.NSK_ERR_UNSUPPORTED
        assert L.nsk_conv2d_dgrad_packed(ctypes.byref(d), ptr(t), ptr(t), ptr(t), 0, st) == B.NSK_ERR_UNSUPPORTED
    assert L.nsk_conv2d_pack_filters(0, None, st) == B.NSK_OK and L.nsk_conv2d_wgrad_reduce(0, None, 0, st) == B.NSK_OK
    assert L.nsk_conv2d_pack_filters(1, None, st) == B.NSK_ERR_NULL and L.nsk_conv2d_wgrad_reduce(-1, None, 0, st) == B.NSK_ERR_BAD_DESC


def test_a_network_bounds_what_its_layers_keep(monkeypatch):
    """Partial sums side by side up to a bound; the layers beyond it give the same gradients through the workspace."""
    units = [dict(kind="conv_bn", name=f"u{i}", src="x" if i == 0 else f"a{i - 1}", dst=f"a{i}", C=32, K=32, R=3, S=3, stride=1, pad=1, relu=True, res=None) for i in range(6)]
    wl = dict(name="six", dtype="bf16", input=(16, 32, 16, 16), units=units, output="a5")
    g = np.random.default_rng(5)
    normal = lambda *s: g.standard_normal(s, dtype=np.float32)
    params = {u["name"]: dict(w=0.08 * normal(32, 32, 3, 3), gamma=1 + 0.1 * normal(32), beta=0.1 * normal(32)) for u in units}
    tensors = dict(x=normal(*wl["input"]), params=params, dout=normal(16, 32, 16, 16))
    d = B.conv_desc(wl["input"], (32, 3, 3), 1, 1, 1, B.NSK_BF16, B.NSK_NHWC)
    one = B.lib().nsk_conv2d_wgrad_partial_bytes(ctypes.byref(d))
    filters = 6 * ((B.lib().nsk_conv2d_packed_filter_bytes(ctypes.byref(d)) + 255) // 256 * 256)
    assert one > 0 and one % 256 == 0 and network.SHARED_SUMS == 64 << 20
    got = []
    for most in (network.SHARED_SUMS, 3 * one, 0):
        monkeypatch.setattr(network, "SHARED_SUMS", most)
        net = network.GpuNetwork(wl, tensors)
        assert net.shared.numel() == max(filters + min(6, most // one) * one, 16)
        net.step()
        torch.cuda.synchronize()
        got.append({k: v.clone() for k, v in net.dw.items()})
    for other in got[1:]:
        assert all(torch.equal(other[k], got[0][k]) for k in got[0])
