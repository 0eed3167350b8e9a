"""The work that libnsk is measured on: layers and blocks of the residual networks, both directions of each, the
grouped layers, a whole training step of the CIFAR-sized network and a step of the recurrent classifier, each
through the calls a training program makes and on buffers it keeps from step to step.

A ``unit`` is one convolution + batch-norm + ReLU (+ shortcut) forward and backward, as GpuNetwork issues it: the
convolution leaves the statistics, the batch-norm leaves the ReLU mask where the layout has one, the shortcut's
gradient is written first and the convolution's gradient is added to it.  Its backward half starts from saved tensors
(convolution output, statistics, mask) that ``prepare`` makes, not from those of the forward half: the ReLU mask of
an element whose pre-activation rounds to either side of zero would otherwise decide a whole gradient element.
"""
import math

import numpy as np
import torch

from paper_2409_11600_amd import binding as B
from paper_2409_11600_amd.network import GpuNetwork
from paper_2409_11600_amd.recurrent import GpuGruClassifier
from paper_2409_11600_amd.trainer import GpuTrainer

DEV = "cuda:0"
EPS = 1e-5


def _unit(name, dtype, N, C, H, W, K, R, stride, residual, layout="nhwc"):
    return dict(name=name, kind="unit", dtype=dtype, layout=layout, N=N, C=C, H=H, W=W, K=K, R=R, stride=stride,
                residual=residual)


def _grouped(name, N, C, H, W, groups, stride, dtype="bf16"):
    return dict(name=name, kind="grouped", dtype=dtype, N=N, C=C, H=H, W=W, groups=groups, stride=stride)


def listed():
    return [
        # the smallest call: one fp32 layer of a small-image network at batch 8, no batch-norm, all three passes
        dict(name="conv_f32_small", kind="conv", dtype="f32", N=8, C=16, H=32, W=32, K=16, R=3, stride=1),
        # second half of the fp32 basic block (fp32 is the storage type of the paper's own runs)
        _unit("unit_f32_block", "f32", 128, 64, 32, 32, 64, 3, 1, True),
        # fp32 in the other layout (NCHW), channel counts and extents that no tile divides
        _unit("unit_f32_nchw_ragged", "f32", 20, 72, 29, 37, 100, 3, 1, False, "nchw"),
        # large-image residual network (ResNet-18 shapes): second convolution of a basic block at 56x56
        _unit("unit_bf16_56", "bf16", 64, 64, 56, 56, 64, 3, 1, True),
        # the strided convolution that enters its second stage
        _unit("unit_bf16_stride2", "bf16", 64, 64, 56, 56, 128, 3, 2, False),
        # its last stage: small image, wide filter
        _unit("unit_bf16_7", "bf16", 64, 512, 7, 7, 512, 3, 1, True),
        # bottleneck blocks: the 1x1 that reduces the large image (the most memory of any layer) ...
        _unit("unit_bf16_reduce", "bf16", 128, 128, 112, 112, 64, 1, 1, False),
        # ... and a 1x1 that widens a small one
        _unit("unit_bf16_expand", "bf16", 128, 256, 14, 14, 1024, 1, 1, False),
        # the image stem: 7x7 stride 2, batch-norm + ReLU, 3x3 max pool
        dict(name="stem_bf16", kind="stem", dtype="bf16", N=64, C=3, H=224, W=224, K=64),
        # a grouped layer, 32 groups of 8 channels
        _grouped("grouped_bf16", 128, 256, 28, 28, 32, 1),
        # whole training step of the CIFAR-sized network with head, loss and optimizer
        dict(name="train_cifar_bf16", kind="train", dtype="bf16", N=256, H=32, W=32, blocks=2, classes=10),
        # step of the recurrent classifier (embedding, GRU, clipped AdamW) at the paper's sizes
        dict(name="gru_f32", kind="gru", dtype="f32", T=200, N=50, V=32768, E=256, H=256, classes=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["unit", "conv", "grouped", "stem", "gru", "train"], [10, 3, 3, 1, 2, 1])[0]
    if kind == "gru":
        return dict(kind=kind, dtype=rng.choice(["f32", "f32", "bf16"]), T=_log(rng, 20, 200), N=_log(rng, 4, 64),
                    V=_log(rng, 1000, 32768), E=8 * _log(rng, 4, 32), H=8 * _log(rng, 4, 32), classes=rng.choice([2, 5, 10]))
    if kind == "train":
        s = rng.choice([24, 28, 32])
        return dict(kind=kind, dtype="bf16", N=_log(rng, 32, 256), H=s, W=s, blocks=rng.choice([1, 2]), classes=rng.choice([10, 100]))
    if kind == "stem":
        return dict(kind=kind, dtype="bf16", N=_log(rng, 4, 64), C=3, H=2 * rng.randint(48, 112), W=2 * rng.randint(48, 112), K=64)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if kind == "grouped":
        per = rng.choice([1, 2, 4, 8, 16])
        groups = _log(rng, 8, 256)
        groups = max(groups - groups % (8 // min(per, 8)), 8)
        s = _log(rng, 7, 56)
        case = dict(kind=kind, dtype=dtype, N=_log(rng, 8, 128), C=per * groups, H=s, W=s + rng.randint(0, 5), groups=groups,
                    stride=rng.choice([1, 1, 2]))
    else:
        R, stride = rng.choice([1, 3, 3]), rng.choice([1, 1, 1, 2])
        step = rng.choice([4, 8, 8, 16])
        C = step * max(1, _log(rng, 16, 1024) // step)
        K = C if rng.random() < 0.5 else step * max(1, _log(rng, 16, 1024) // step)
        s = _log(rng, 7, 112)
        case = dict(kind=kind, dtype=dtype, N=_log(rng, 1, 128), C=C, H=s, W=max(7, s + rng.randint(-4, 4)), K=K, R=R, stride=stride)
        if kind == "unit":
            case["residual"] = bool(stride == 1 and C == K and rng.random() < 0.7)
            case["layout"] = rng.choice(["nhwc", "nhwc", "nhwc", "nchw"])
    # no larger than the largest listed layer: fewer images where a draw would be
    while case["N"] > 1 and (work(case)["flops"] > (9e10 if dtype == "bf16" else 3e10) or work(case)["bytes"] > 8e8):
        case["N"] //= 2
    while case.get("H", 0) > 14 and (work(case)["flops"] > (9e10 if dtype == "bf16" else 3e10) or work(case)["bytes"] > 8e8):
        case["H"], case["W"] = case["H"] // 2, case["W"] // 2
    return case


# ------------------------------------------------------------------------------------------------ sizes

def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _es(case):
    return 2 if case["dtype"] == "bf16" else 4


def _layout(case):
    return B.NSK_NCHW if case.get("layout") == "nchw" else B.NSK_NHWC


def _geometry(case):
    """(K, R, stride, pad, P, Q, channels per group) of the case's convolution."""
    R = case.get("R", 7 if case["kind"] == "stem" else 3)
    stride = case.get("stride", 2)
    pad = R // 2
    K = case.get("K", case["C"])
    out = lambda n: (n + 2 * pad - R) // stride + 1
    return K, R, stride, pad, out(case["H"]), out(case["W"]), case["C"] // case.get("groups", 1)


def _cifar_units(blocks):
    """Stem and three stages of basic blocks (16, 32, 64 channels), the later two entered with stride 2."""
    units = []

    def conv(name, src, dst, C, K, R, stride, relu=True, res=None):
        units.append(dict(kind="conv_bn", name=name, src=src, dst=dst, C=C, K=K, R=R, S=R, stride=stride, pad=R // 2, relu=relu, res=res))

    conv("stem", "x", "s0", 3, 16, 3, 1)
    src, C = "s0", 16
    for s, K in enumerate((16, 32, 64)):
        for b in range(blocks):
            dst, stride = f"s{s + 1}b{b + 1}", 2 if b == 0 and K != C else 1
            conv(dst + ".c1", src, dst + ".a", C, K, 3, stride)
            res = src
            if stride != 1:
                res = dst + ".sc"
                conv(dst + ".proj", src, res, C, K, 1, stride, relu=False)
            conv(dst + ".c2", dst + ".a", dst, K, K, 3, 1, res=res)
            src, C = dst, K
    return units


def _workload(case):
    units = _cifar_units(case["blocks"])
    return dict(name="cifar", dtype=case["dtype"], input=(case["N"], 3, case["H"], case["W"]), units=units, output=units[-1]["dst"])


def work(case):
    """What one pass cannot do without: every input read once, every output and saved tensor written once."""
    es, kind = _es(case), case["kind"]
    if kind == "gru":
        T, N, V, E, H, K = (case[k] for k in ("T", "N", "V", "E", "H", "classes"))
        weights = V * E + 3 * H * (E + H + 2) + K * (H + 1)
        return dict(flops=3 * 2 * T * N * 3 * H * (E + H) + 3 * 2 * N * H * K,
                    bytes=6 * 4 * weights + T * N * (2 * E + 9 * H) * es + 4 * T * N)
    if kind == "train":
        flops = bytes_ = 0
        hw = {"x": (case["H"], case["W"])}
        for u in _cifar_units(case["blocks"]):
            h, w = hw[u["src"]]
            p, q = (h - 1) // u["stride"] + 1, (w - 1) // u["stride"] + 1
            hw[u["dst"]] = (p, q)
            flops += 3 * 2 * case["N"] * p * q * u["K"] * u["C"] * u["R"] ** 2
            weights = u["K"] * u["C"] * u["R"] ** 2 + 2 * u["K"]
            # forward: x read, y and out written; backward: x, y and dout read, dx written
            bytes_ += case["N"] * (3 * h * w * u["C"] + 4 * p * q * u["K"]) * es + weights * 4 * 6
        return dict(flops=flops, bytes=bytes_)
    K, R, _, _, P, Q, cg = _geometry(case)
    x, y, w = case["N"] * case["C"] * case["H"] * case["W"], case["N"] * K * P * Q, K * cg * R * R
    flops = 3 * 2 * y * cg * R * R
    if kind in ("conv", "grouped"):
        return dict(flops=flops, bytes=(2 * x + 2 * y + 2 * w) * es + 4 * w)
    if kind == "stem":
        pooled = case["N"] * K * ((P - 1) // 2 + 1) * ((Q - 1) // 2 + 1)
        return dict(flops=flops, bytes=(2 * x + 3 * y + 2 * w + 2 * pooled) * es + 2 * pooled + 4 * w)
    return dict(flops=flops, bytes=(2 * x + (4 + int(case["residual"])) * y + 2 * w) * es + 4 * w)


# ------------------------------------------------------------------------------------------------ inputs

def _generator(seed, device=DEV):
    return torch.Generator(device=device).manual_seed(int(seed))


def _activation(case, g, C, H, W, scale=1.0):
    shape = (case["N"], C, H, W) if _layout(case) == B.NSK_NCHW else (case["N"], H, W, C)
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(scale).to(_dtype(case))


def _filter(case, g):
    K, R, _, _, _, _, cg = _geometry(case)
    shape = (K, cg, R, R) if _layout(case) == B.NSK_NCHW else (K, R, R, cg)
    return (torch.randn(shape, generator=g, device=DEV) * math.sqrt(2.0 / (cg * R * R))).to(_dtype(case))


def _inputs(case, seed):
    """Inputs of a layer (and of its batch-norm), all on the device."""
    g = _generator(seed)
    K, R, stride, pad, P, Q, cg = _geometry(case)
    s = dict(case=case, x=_activation(case, g, case["C"], case["H"], case["W"]), w=_filter(case, g))
    if case["kind"] in ("conv", "grouped"):
        s["dout"] = _activation(case, g, K, P, Q)
        return s
    s["gamma"] = 1.0 + 0.2 * torch.randn(K, generator=g, device=DEV)
    s["beta"] = 0.2 * torch.randn(K, generator=g, device=DEV)
    s["residual"] = _activation(case, g, K, P, Q) if case.get("residual") else None
    # what a forward pass has left for the backward pass: the convolution's output, its statistics, the activation
    s["y_saved"] = _activation(case, g, K, P, Q, 1.3)
    axes = (0, 2, 3) if _layout(case) == B.NSK_NCHW else (0, 1, 2)
    n = case["N"] * P * Q
    per = [-1 if a not in axes else 1 for a in range(4)]
    total = s["y_saved"].sum(axes, dtype=torch.float32).double() / n
    square = (s["y_saved"].float() ** 2).sum(axes).double() / n
    s["mean_saved"], s["invstd_saved"] = total.float(), torch.rsqrt((square - total * total).clamp_min(0) + EPS).float()
    z = (s["y_saved"].float() - s["mean_saved"].view(per)) * (s["invstd_saved"] * s["gamma"]).view(per) + s["beta"].view(per)
    if s["residual"] is not None:
        z += s["residual"]
    s["out_saved"] = z.clamp_min_(0).to(_dtype(case))
    if case["kind"] == "stem":
        pp, pq = (P - 1) // 2 + 1, (Q - 1) // 2 + 1
        s["dout"] = _activation(case, g, K, pp, pq)
        # the place (r*3 + s) of each window's maximum: any place inside the image is a possible one
        idx = torch.randint(0, 9, s["dout"].shape, generator=g, device=DEV, dtype=torch.int8)
        r, c = torch.div(idx, 3, rounding_mode="floor"), idx % 3
        h = torch.arange(pp, device=DEV, dtype=torch.int16).view(1, pp, 1, 1) * 2 - 1 + r
        v = torch.arange(pq, device=DEV, dtype=torch.int16).view(1, 1, pq, 1) * 2 - 1 + c
        s["idx_saved"] = torch.where((h >= 0) & (h < P) & (v >= 0) & (v < Q), idx, torch.full_like(idx, 4)).contiguous()
    else:
        s["dout"] = _activation(case, g, K, P, Q)
    return s


def _mask(out, nbytes):
    """One byte per 16-byte vector of `out`, bit e set where element e is above zero."""
    per = 16 // out.element_size()
    bits = torch.tensor([1 << e for e in range(per)], dtype=torch.float32, device=out.device)
    mask = torch.mv((out.reshape(-1, per) > 0).float(), bits).to(torch.uint8)
    assert mask.numel() == nbytes
    return mask


def _network_tensors(case, seed, wl):
    g = np.random.default_rng(seed)
    normal = lambda shape, std=1.0: (g.standard_normal(shape, dtype=np.float32) * np.float32(std))
    rounded = lambda a: torch.from_numpy(a).to(_dtype(case)).float().numpy()
    params = {}
    for u in wl["units"]:
        w = normal((u["K"], u["C"], u["R"], u["S"]), math.sqrt(2.0 / (u["C"] * u["R"] ** 2)))
        params[u["name"]] = dict(w=rounded(w), gamma=1 + normal(u["K"], 0.2), beta=normal(u["K"], 0.2))
    s = case["H"]
    for _ in range(2):
        s = (s - 1) // 2 + 1
    return dict(x=rounded(g.random(wl["input"], dtype=np.float32)), params=params, dout=np.zeros((case["N"], 64, s, s), np.float32),
                fc_w=normal((case["classes"], 64), 0.125), fc_b=normal(case["classes"], 0.1),
                labels=g.integers(0, case["classes"], case["N"]).astype(np.int32))


def _gru_arrays(case, seed):
    g = np.random.default_rng(seed)
    T, N, V, E, H, K = (case[k] for k in ("T", "N", "V", "E", "H", "classes"))
    uniform = lambda *shape: ((g.random(shape, dtype=np.float32) * 2 - 1) / np.float32(math.sqrt(H)))
    return dict(tokens=g.integers(0, V, (T, N)).astype(np.int32), labels=g.integers(0, K, N).astype(np.int32),
                table=g.standard_normal((V, E), dtype=np.float32), w_ih=uniform(3 * H, E), w_hh=uniform(3 * H, H),
                b_ih=uniform(3 * H), b_hh=uniform(3 * H), w_out=uniform(K, H), b_out=uniform(K))


LR = 0.02


def prepare(case, seed):
    kind, dt = case["kind"], _dtype(case)
    if kind == "train":
        wl = _workload(case)
        t = _network_tensors(case, seed, wl)
        return dict(case=case, trainer=GpuTrainer(GpuNetwork(wl, t, device=DEV), t["fc_w"], t["fc_b"], t["labels"], lr=LR))
    if kind == "gru":
        return dict(case=case, model=GpuGruClassifier(dtype=case["dtype"], device=DEV, **_gru_arrays(case, seed)))
    s = _inputs(case, seed)
    K, R, stride, pad, P, Q, cg = _geometry(case)
    lay = _layout(case)
    s["ws"] = B.Workspace(DEV)
    s["dw"] = torch.empty(s["w"].shape, dtype=torch.float32, device=DEV)
    s["dx"] = torch.empty_like(s["x"])
    shape = B._act_shape(case["N"], K, P, Q, lay)
    s["y"] = torch.empty(shape, dtype=dt, device=DEV)
    if kind in ("conv", "grouped"):
        return s
    d = B.conv_desc((case["N"], case["C"], case["H"], case["W"]), (K, R, R), stride, pad, 1, B._dtype_code(s["x"]), lay)
    s["stats"] = torch.empty((2, int(B.nsk_conv2d_stats_rows(d)), K), dtype=torch.float32, device=DEV)
    s["out"], s["dy"] = torch.empty_like(s["y"]), torch.empty_like(s["y"])
    for name in ("mean", "invstd", "dgamma", "dbeta"):
        s[name] = torch.empty(K, dtype=torch.float32, device=DEV)
    nbytes = B.bn_mask_bytes(s["y"], lay)
    s["mask"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None
    s["mask_saved"] = _mask(s["out_saved"], nbytes) if nbytes else None
    if nbytes:
        s["out_saved"] = None
    if kind == "stem":
        s["pooled"], s["idx"] = torch.empty_like(s["dout"]), torch.empty(s["dout"].shape, dtype=torch.int8, device=DEV)
        s["dpool"] = torch.empty_like(s["y"])
    return s


# ------------------------------------------------------------------------------------------------ one pass

def _run_layer(s):
    case = s["case"]
    _, R, stride, pad, _, _, cg = _geometry(case)
    K, dims = s["w"].shape[0], (case["N"], case["C"], case["H"], case["W"])
    if case["kind"] == "grouped":
        G = case["groups"]
        B.conv2d_grouped_fwd(s["x"], s["w"], G, stride, pad, out=s["y"], ws=s["ws"])
        B.conv2d_grouped_wgrad(s["x"], s["dout"], (K, cg, R, R), G, stride, pad, out=s["dw"], ws=s["ws"])
        B.conv2d_grouped_dgrad(s["dout"], s["w"], dims, G, stride, pad, out=s["dx"], ws=s["ws"])
    else:
        B.conv2d_fwd(s["x"], s["w"], stride, pad, out=s["y"], ws=s["ws"])
        B.conv2d_wgrad(s["x"], s["dout"], (K, cg, R, R), stride, pad, out=s["dw"], ws=s["ws"])
        B.conv2d_dgrad(s["dout"], s["w"], dims, stride, pad, out=s["dx"], ws=s["ws"])
    return dict(y=s["y"], dw=s["dw"], dx=s["dx"])


def _run_unit(s):
    case, lay, ws = s["case"], _layout(s["case"]), s["ws"]
    K, R, stride, pad, _, _, cg = _geometry(case)
    dims = (case["N"], case["C"], case["H"], case["W"])
    stem, shortcut = case["kind"] == "stem", s["residual"] is not None
    # forward
    B.conv2d_fwd_stats(s["x"], s["w"], stride, pad, layout=lay, out=s["y"], stats=s["stats"], ws=ws)
    B.bn_relu_add_fwd(s["y"], s["gamma"], s["beta"], s["residual"], eps=EPS, layout=lay, out=s["out"], save_mean=s["mean"],
                      save_invstd=s["invstd"], ws=ws, relu_mask=s["mask"], stats=s["stats"])
    dout = s["dout"]
    if stem:
        B.maxpool2d_fwd(s["out"], out=s["pooled"], idx=s["idx"])
        dout = B.maxpool2d_bwd(dout, s["idx_saved"], tuple(s["out"].shape[i] for i in (0, 3, 1, 2)), out=s["dpool"])
    # backward: the shortcut's gradient goes straight to where the convolution's is added
    B.bn_relu_add_bwd(s["y_saved"], s["out_saved"], dout, s["gamma"], s["mean_saved"], s["invstd_saved"], layout=lay, eps=EPS,
                      dx=s["dy"], dresidual=s["dx"] if shortcut else None, dgamma=s["dgamma"], dbeta=s["dbeta"], ws=ws,
                      relu_mask=s["mask_saved"])
    B.conv2d_wgrad(s["x"], s["dy"], (K, cg, R, R), stride, pad, layout=lay, out=s["dw"], ws=ws)
    B.conv2d_dgrad(s["dy"], s["w"], dims, stride, pad, layout=lay, out=s["dx"], accumulate=shortcut, ws=ws)
    got = {k: s[k] for k in ("y", "out", "mean", "invstd", "dy", "dgamma", "dbeta", "dw", "dx")}
    if stem:
        got.update(pooled=s["pooled"], idx=s["idx"], dpool=s["dpool"])
    return got


def run(s):
    kind = s["case"]["kind"]
    if kind in ("conv", "grouped"):
        return _run_layer(s)
    if kind in ("unit", "stem"):
        return _run_unit(s)
    if kind == "train":
        t = s["trainer"]
        t.step()
        got = dict(loss=t.loss, logits=t.logits, fc_w=t.fc_w_master, fc_b=t.fc_b)
        for name in t.master:
            got["w." + name], got["gamma." + name], got["beta." + name] = t.master[name], t.net.gamma[name], t.net.beta[name]
        return got
    m = s["model"]
    m.step()
    return dict(loss=m.loss, logits=m.logits, **m.master)


# ------------------------------------------------------------------------------------------------ how close

def tolerance(case):
    # measured against `exact` over the listed and drawn cases, times about four
    kind, dtype = case["kind"], case["dtype"]
    if kind == "train":
        return dict(rel=2e-2, max=0.1)
    if kind == "gru":
        # the first step of AdamW moves every weight by lr times the sign of its gradient, also where that is nearly 0
        return dict(rel=2e-5, max=1e-2) if dtype == "f32" else dict(rel=2e-2, max=0.1)
    if dtype == "f32":
        return dict(rel=5e-6, max=4e-5)
    # one rounding to bf16 a stored tensor; idx: ties of the pool's windows after it
    return dict(rel=7e-3, max=5e-2, differ=5e-3) if kind == "stem" else dict(rel=7e-3, max=5e-2)


# The same in 64 bits, a product per filter tap.  What is stored in bf16 between two calls is rounded to bf16 here too:
# the next call is defined on the stored values.

def _taps(n, out, R, stride, pad, r):
    """Output positions whose tap r lies in the image, and the image positions it lies on."""
    lo = max(0, -(-(pad - r) // stride))
    hi = min(out, (n - 1 + pad - r) // stride + 1)
    return (slice(lo, hi), slice(lo * stride - pad + r, (hi - 1) * stride - pad + r + 1, stride)) if hi > lo else None


def _each_tap(H, W, P, Q, R, stride, pad):
    for r in range(R):
        for c in range(R):
            a, b = _taps(H, P, R, stride, pad, r), _taps(W, Q, R, stride, pad, c)
            if a and b:
                yield r, c, (slice(None), a[0], b[0]), (slice(None), a[1], b[1])


def _conv64(x, w, stride, pad, groups=1):
    """NHWC, KRSC."""
    N, H, W, C = x.shape
    K, R, _, cg = w.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    y = torch.zeros((N, P, Q, K), dtype=torch.float64, device=x.device)
    kg = K // groups
    for r, c, o, i in _each_tap(H, W, P, Q, R, stride, pad):
        xs = x[i]
        if groups == 1:
            y[o] += (xs.reshape(-1, C) @ w[:, r, c].t()).view(xs.shape[:3] + (K,))
        else:
            ys = y[o].view(xs.shape[:3] + (groups, kg))
            xg, wg = xs.reshape(xs.shape[:3] + (groups, cg)), w[:, r, c].reshape(groups, kg, cg)
            for ci in range(cg):
                ys += xg[..., ci:ci + 1] * wg[..., ci]
            y[o] = ys.view(xs.shape[:3] + (K,))
    return y


def _dgrad64(dy, w, x_shape, stride, pad, groups=1):
    N, H, W, C = x_shape
    K, R, _, cg = w.shape
    P, Q = dy.shape[1:3]
    dx = torch.zeros(x_shape, dtype=torch.float64, device=dy.device)
    kg = K // groups
    for r, c, o, i in _each_tap(H, W, P, Q, R, stride, pad):
        ds = dy[o]
        if groups == 1:
            dx[i] += (ds.reshape(-1, K) @ w[:, r, c]).view(ds.shape[:3] + (C,))
        else:
            dg, wg = ds.reshape(ds.shape[:3] + (groups, kg)), w[:, r, c].reshape(groups, kg, cg)
            add = torch.zeros(ds.shape[:3] + (groups, cg), dtype=torch.float64, device=dy.device)
            for ki in range(kg):
                add += dg[..., ki:ki + 1] * wg[:, ki]
            dx[i] += add.view(ds.shape[:3] + (C,))
    return dx


def _wgrad64(x, dy, R, stride, pad, groups=1):
    N, H, W, C = x.shape
    P, Q, K = dy.shape[1:]
    cg, kg = C // groups, K // groups
    dw = torch.zeros((K, R, R, cg), dtype=torch.float64, device=x.device)
    for r, c, o, i in _each_tap(H, W, P, Q, R, stride, pad):
        xs, ds = x[i], dy[o]
        if groups == 1:
            dw[:, r, c] = ds.reshape(-1, K).t() @ xs.reshape(-1, C)
        else:
            xg, dg = xs.reshape(-1, groups, cg), ds.reshape(-1, groups, kg)
            for ki in range(kg):
                for ci in range(cg):
                    dw[:, r, c].view(groups, kg, cg)[:, ki, ci] = (dg[:, :, ki] * xg[:, :, ci]).sum(0)
    return dw


def _bn64(y, gamma, beta, residual, relu=True):
    mean = y.mean((0, 1, 2))
    invstd = torch.rsqrt(((y - mean) ** 2).mean((0, 1, 2)) + EPS)
    z = (y - mean) * (invstd * gamma) + beta
    if residual is not None:
        z = z + residual
    return (z.clamp_min(0) if relu else z), mean, invstd


def _bn_bwd64(y, dz, gamma, mean, invstd):
    xhat = (y - mean) * invstd
    dbeta, dgamma = dz.sum((0, 1, 2)), (dz * xhat).sum((0, 1, 2))
    n = dz.numel() // dz.shape[-1]
    return gamma * invstd * (dz - dbeta / n - xhat * (dgamma / n)), dgamma, dbeta


def _pool64(x):
    """3x3 windows, stride 2, padding 1: the maxima and the first place of each."""
    N, H, W, C = x.shape
    P, Q = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    best = torch.full((N, P, Q, C), -math.inf, dtype=x.dtype, device=x.device)
    place = torch.full((N, P, Q, C), -1, dtype=torch.int8, device=x.device)
    for r, c, o, i in _each_tap(H, W, P, Q, 3, 2, 1):
        more = x[i] > best[o]
        best[o] = torch.where(more, x[i], best[o])
        place[o] = torch.where(more, torch.full_like(place[o], 3 * r + c), place[o])
    return best, place


def _pool_bwd64(dy, place, shape):
    dx = torch.zeros(shape, dtype=torch.float64, device=dy.device)
    for r, c, o, i in _each_tap(shape[1], shape[2], dy.shape[1], dy.shape[2], 3, 2, 1):
        dx[i] += torch.where(place[o] == 3 * r + c, dy[o], torch.zeros((), dtype=torch.float64, device=dy.device))
    return dx


def _exact_layer(case, seed):
    s = _inputs(case, seed)
    nchw = _layout(case) == B.NSK_NCHW
    inner = lambda t: (t.permute(0, 2, 3, 1) if nchw else t).double().contiguous()
    outer = lambda t: t.permute(0, 3, 1, 2).contiguous() if nchw else t
    stored = lambda t: t.to(_dtype(case)).double()
    _, R, stride, pad, _, _, _ = _geometry(case)
    G = case.get("groups", 1)
    x, w = inner(s["x"]), inner(s["w"])
    y = _conv64(x, w, stride, pad, G)
    if case["kind"] in ("conv", "grouped"):
        dout = inner(s["dout"])
        return dict(y=outer(y), dw=outer(_wgrad64(x, dout, R, stride, pad, G)), dx=outer(_dgrad64(dout, w, x.shape, stride, pad, G)))
    gamma, beta = s["gamma"].double(), s["beta"].double()
    residual = inner(s["residual"]) if s["residual"] is not None else None
    out, mean, invstd = _bn64(stored(y), gamma, beta, residual)
    got = dict(y=outer(y), out=outer(out), mean=mean, invstd=invstd)
    dout = inner(s["dout"])
    if case["kind"] == "stem":
        pooled, place = _pool64(stored(out))
        dpool = _pool_bwd64(dout, s["idx_saved"], tuple(out.shape))
        got.update(pooled=pooled, idx=None, dpool=dpool)
        dout = stored(dpool)
    dz = torch.where(inner(s["out_saved"]) > 0, dout, torch.zeros((), dtype=torch.float64, device=DEV))
    dy, dgamma, dbeta = _bn_bwd64(inner(s["y_saved"]), dz, gamma, s["mean_saved"].double(), s["invstd_saved"].double())
    got.update(dy=outer(dy), dgamma=dgamma, dbeta=dbeta)
    dy = stored(dy)
    dx = _dgrad64(dy, w, x.shape, stride, pad)
    if residual is not None:
        dx = dx + dz
    got.update(dw=outer(_wgrad64(x, dy, R, stride, pad)), dx=outer(dx))
    return got


def _exact_train(case, seed):
    wl = _workload(case)
    t = _network_tensors(case, seed, wl)
    dev = lambda a: torch.from_numpy(a).to(DEV).double()
    stored = lambda a: a.to(_dtype(case)).double()
    act, saved = {"x": dev(t["x"]).permute(0, 2, 3, 1).contiguous()}, {}
    for u in wl["units"]:
        p = t["params"][u["name"]]
        w, gamma, beta = dev(p["w"]).permute(0, 2, 3, 1).contiguous(), dev(p["gamma"]), dev(p["beta"])
        y = stored(_conv64(act[u["src"]], w, u["stride"], u["pad"]))
        out, mean, invstd = _bn64(y, gamma, beta, act[u["res"]] if u["res"] else None, u["relu"])
        act[u["dst"]] = stored(out)
        saved[u["name"]] = (w, gamma, beta, y, mean, invstd)
    top = act[wl["output"]]
    pooled = stored(top.mean((1, 2)))
    fc_w, fc_b = dev(t["fc_w"]), dev(t["fc_b"])
    logits = stored(stored(pooled @ stored(fc_w).t()) + fc_b)
    rows = torch.arange(case["N"], device=DEV)
    labels = torch.from_numpy(t["labels"]).to(DEV).long()
    loss = (torch.logsumexp(logits, 1) - logits[rows, labels]).mean()
    d = torch.softmax(logits, 1)
    d[rows, labels] -= 1
    d = stored(d / case["N"])
    step = lambda w, g, decay: w - LR * (g + decay * w)
    got = dict(loss=loss.view(1), logits=logits, fc_w=step(fc_w, d.t() @ pooled, 1e-4), fc_b=step(fc_b, d.sum(0), 0.0))
    dtop = stored(stored(d @ stored(fc_w)) / (top.shape[1] * top.shape[2]))
    grad = {wl["output"]: dtop[:, None, None, :].expand(top.shape).contiguous()}
    for u in reversed(wl["units"]):
        name = u["name"]
        w, gamma, beta, y, mean, invstd = saved[name]
        dz = grad[u["dst"]]
        if u["relu"]:
            dz = torch.where(act[u["dst"]] > 0, dz, torch.zeros((), dtype=torch.float64, device=DEV))
        if u["res"]:
            grad[u["res"]] = dz
        dy, dgamma, dbeta = _bn_bwd64(y, dz, gamma, mean, invstd)
        dy = stored(dy)
        dx = _dgrad64(dy, w, act[u["src"]].shape, u["stride"], u["pad"])
        grad[u["src"]] = stored(grad[u["src"]] + dx if u["src"] in grad else dx)
        got["w." + name] = step(w, _wgrad64(act[u["src"]], dy, u["R"], u["stride"], u["pad"]), 1e-4)
        got["gamma." + name], got["beta." + name] = step(gamma, dgamma, 0.0), step(beta, dbeta, 0.0)
    return got


def _exact_gru(case, seed):
    if case["dtype"] == "bf16":
        return None      # every step of the sequence rounds its state and gates: no one value
    a = _gru_arrays(case, seed)
    p = {k: torch.from_numpy(a[k]).to(DEV).double().requires_grad_() for k in ("table", "w_ih", "w_hh", "w_out", "b_ih", "b_hh", "b_out")}
    tokens, labels = torch.from_numpy(a["tokens"]).to(DEV).long(), torch.from_numpy(a["labels"]).to(DEV).long()
    H = case["H"]
    x = torch.nn.functional.embedding(tokens, p["table"])
    gi = x.reshape(-1, case["E"]) @ p["w_ih"].t() + p["b_ih"]
    gi = gi.view(case["T"], case["N"], 3 * H)
    h = torch.zeros((case["N"], H), dtype=torch.float64, device=DEV)
    for t in range(case["T"]):
        gh = h @ p["w_hh"].t() + p["b_hh"]
        r, z = torch.sigmoid(gi[t, :, :H] + gh[:, :H]), torch.sigmoid(gi[t, :, H:2 * H] + gh[:, H:2 * H])
        n = torch.tanh(gi[t, :, 2 * H:] + r * gh[:, 2 * H:])
        h = (1 - z) * n + z * h
    logits = h @ p["w_out"].t() + p["b_out"]
    loss = torch.nn.functional.cross_entropy(logits, labels)
    loss.backward()
    norm = torch.sqrt(sum((v.grad ** 2).sum() for v in p.values()))
    scale = min(1.0, 5.0 / (float(norm) + 1e-6))
    got = dict(loss=loss.detach().view(1), logits=logits.detach())
    for k, v in p.items():
        g, w = v.grad * scale, v.detach()
        w = w * (1 - 1e-3 * (0.0 if k.startswith("b_") else 1e-4))
        m, q = 0.1 * g / (1 - 0.9), 0.001 * g * g / (1 - 0.999)
        got[k] = w - 1e-3 * m / (torch.sqrt(q) + 1e-8)
    return got


def exact(case, seed):
    kind = case["kind"]
    with torch.enable_grad() if kind == "gru" else torch.no_grad():
        return _exact_train(case, seed) if kind == "train" else _exact_gru(case, seed) if kind == "gru" else _exact_layer(case, seed)
