"""All GRU steps in one call: every instance of the sequence kernel (hidden sizes 64, 128, 192, 256 and ragged ones below), one
sample and several, one step and several, and the sizes above it that run step by step, against the oracle's gates and
products on the values as stored."""
import numpy as np
import pytest
import torch

import nsk_inputs as gen
from oracle import gru as G
from paper_2409_11600_amd import binding as B
from parity import TOL, guarded, max_rel_err, on_grid, torch_dtype

pytestmark = pytest.mark.gpu


def dev(a, dtype="f32"):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda:0", dtype=torch_dtype(dtype))


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,N,H", [(1, 2, 8), (5, 1, 64), (4, 3, 72), (3, 2, 128), (4, 2, 168), (3, 1, 192), (4, 2, 200), (5, 3, 256), (3, 2, 264)])
def test_sequence_calls(T, N, H, dtype):
    print(f"gru sequence T={T} N={N} H={H} {dtype}", flush=True)
    s, tol = 8800 + H, TOL[dtype]
    gi = on_grid(gen.normal(s, 0, (T, N, 3 * H)), dtype)
    w = on_grid(gen.normal(s, 1, (3 * H, H)) / np.sqrt(H), dtype)
    b_ih, b_hh = (0.3 * gen.normal(s, 2 + k, (3 * H,)).astype(np.float32) for k in range(2))
    h0, dh_top = (on_grid(gen.normal(s, 4 + k, (N, H)), dtype) for k in range(2))
    stored = lambda a: on_grid(np.asarray(a, np.float32), dtype).astype(np.float64)
    dt = torch_dtype(dtype)
    h, h_ok = guarded((T + 1, N, H), dt)
    saved, s_ok = guarded((T, N, 4 * H), dt)
    h[0] = dev(h0, dtype)
    B.gru_seq_fwd(dev(gi, dtype), dev(w, dtype), dev(b_ih), dev(b_hh), h, saved)
    torch.cuda.synchronize()
    h_ok(), s_ok()
    gh, gs = host(h), host(saved)
    w64 = w.astype(np.float64)
    hp = h0.astype(np.float64)
    for t in range(T):
        hn, r, z, n, q = G.gru_gates_fwd(gi[t], hp @ w64.T, b_ih, b_hh, hp)
        assert max_rel_err(gh[t + 1], hn) <= tol
        for k, want in enumerate((r, z, n, q)):
            assert max_rel_err(gs[t][:, k * H:(k + 1) * H], want) <= tol
        hp = gh[t + 1]                      # each step is held to the bar on the state as stored
    outs = [guarded((T, N, 3 * H), dt) for _ in range(2)]
    scratch = torch.empty((2, N, H), dtype=dt, device="cuda:0")
    B.gru_seq_bwd(saved, h, dev(dh_top, dtype), dev(w.T, dtype), outs[0][0], outs[1][0], scratch)
    torch.cuda.synchronize()
    for _, ok in outs:
        ok()
    dgi, dgh = host(outs[0][0]), host(outs[1][0])
    dh = dh_top.astype(np.float64)
    for t in reversed(range(T)):
        r, z, n, q = (gs[t][:, k * H:(k + 1) * H] for k in range(4))
        wgi, wgh, direct = G.gru_gates_bwd(r, z, n, q, gh[t], dh)
        assert max_rel_err(dgi[t], wgi) <= tol
        assert max_rel_err(dgh[t], wgh) <= tol
        dh = stored(direct) + dgh[t] @ w64
    # the step calls, one by one, give the same to rounding
    hs, hp = [], dev(h0, dtype)
    for t in range(T):
        hp, _ = B.gru_step_fwd(dev(gi[t], dtype), dev(w, dtype), dev(b_ih), dev(b_hh), hp)
        hs.append(host(hp))
    assert max_rel_err(gh[1:], np.stack(hs)) <= T * tol


def test_sequence_calls_refuse_what_the_step_calls_refuse():
    z = lambda *s: torch.zeros(s, device="cuda:0")
    with pytest.raises(B.NskError) as e:     # too many rows
        B.gru_seq_fwd(z(2, 300, 24), z(24, 8), z(24), z(24), z(3, 300, 8), z(2, 300, 32))
    assert e.value.status == B.NSK_ERR_UNSUPPORTED
    with pytest.raises(B.NskError) as e:     # the second step's rows are not on a 16-byte boundary
        zb = lambda *s: torch.zeros(s, device="cuda:0", dtype=torch.bfloat16)
        B.gru_seq_fwd(zb(2, 1, 12), zb(12, 4), z(12), z(12), zb(3, 1, 4), zb(2, 1, 16))
    assert e.value.status == B.NSK_ERR_ALIGNMENT


def _sequence(T, N, H, dtype, seed, bad=None):
    """Operands of both calls and a function that makes the calls; `bad`: a value for one element of the initial state."""
    dt = torch_dtype(dtype)
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    r = lambda *s, k=1.0: (torch.randn(s, generator=g, device="cuda:0") * k).to(dt)
    gi, w, h0, top = r(T, N, 3 * H), r(3 * H, H, k=H ** -0.5), r(N, H), r(N, H)
    b = [0.3 * torch.randn(3 * H, generator=g, device="cuda:0") for _ in range(2)]
    wt = w.t().contiguous()
    if bad is not None:
        h0[0, 1] = bad
    h, saved = torch.empty((T + 1, N, H), dtype=dt, device="cuda:0"), torch.empty((T, N, 4 * H), dtype=dt, device="cuda:0")
    h[0] = h0
    dgi, dgh = (torch.empty((T, N, 3 * H), dtype=dt, device="cuda:0") for _ in range(2))
    scratch = torch.empty((2, N, H), dtype=dt, device="cuda:0")

    def run():
        B.gru_seq_fwd(gi, w, *b, h, saved)
        B.gru_seq_bwd(saved, h, top, wt, dgi, dgh, scratch)

    return run, (h, saved, dgi, dgh)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,N,H", [(1, 2, 256), (2, 1, 200), (7, 9, 256), (3, 64, 248), (16, 65, 208), (16, 128, 256), (15, 128, 256), (1, 70, 256), (16, 129, 256)])
def test_blocks_that_share_a_sample(T, N, H, dtype, nsk_env):
    """Several blocks per sample (as many as the sizes allow, and at most two) add in the order of one: the same bits.  Sizes:
    a step without an exchange, part of a last block, all eight XCDs full at four and at two blocks, and one sample more."""
    print(f"gru split T={T} N={N} H={H} {dtype}", flush=True)
    run, out = _sequence(T, N, H, dtype, 8900 + H)
    blocks = lambda: B.gru_seq_blocks(torch_dtype(dtype), T, N, H)
    nsk_env("NSK_GRU_SPLIT", "1")
    assert blocks() == 1
    run()
    want = [o.clone() for o in out]
    for most in (None, "2"):
        nsk_env("NSK_GRU_SPLIT", most)
        # (the route that is meant is the one that runs: bf16 samples are not shared by two)
        two = 1 if dtype == "bf16" or N > 128 or 1 < T < 16 else 2
        assert blocks() == (4 if N <= 64 and most is None else two)
        for o in (out[0][1:], *out[1:]):
            o.zero_()
        run()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))


def test_sizes_that_are_not_shared():
    blocks = lambda N, H, dt=torch.float32: B.gru_seq_blocks(dt, 20, N, H)
    assert blocks(50, 192) == blocks(50, 252) == blocks(50, 64, torch.bfloat16) == 1     # the weight fits a CU; rows of no whole 8-byte words
    assert blocks(50, 260) == blocks(300, 256) == 0                                     # step launches; refused


@pytest.mark.parametrize("polls", ["0", "3", "40"])
@pytest.mark.parametrize("dtype,T,N,H", [("f32", 9, 50, 256), ("f32", 17, 70, 200), ("bf16", 9, 33, 256), ("bf16", 2, 3, 224), ("f32", 1, 3, 256)])
def test_blocks_that_give_up_waiting(dtype, T, N, H, polls, nsk_env):
    """A block that has waited too long ends (with a bound of 0 polls every block does, at its second step; with 3 and 40 some do, some
    later, some never), and the call still gives every sample what one block computes: the same bits."""
    print(f"gru give-up T={T} N={N} H={H} {dtype} polls={polls}", flush=True)
    run, out = _sequence(T, N, H, dtype, 8910 + H)
    nsk_env("NSK_GRU_SPLIT", "1")
    run()
    want = [o.clone() for o in out]
    nsk_env("NSK_GRU_SPLIT", None)
    nsk_env("NSK_GRU_POLLS", polls)
    assert B.gru_seq_blocks(torch_dtype(dtype), T, N, H) > 1
    for _ in range(3):
        for o in (out[0][1:], *out[1:]):
            o.zero_()
        run()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_blocks_that_share_a_sample_with_nan(dtype):
    """A state that holds the very NaN that stands for "not there yet" (all ones), and infinity: the calls end, the sample's later
    states hold NaN, the other samples' values are those without it."""
    T, N, H = 3, 3, 256
    assert B.gru_seq_blocks(torch_dtype(dtype), T, N, H) == 4
    run, clean = _sequence(T, N, H, dtype, 8901)
    run()
    ones = torch.tensor([-1], dtype=torch.int32 if dtype == "f32" else torch.int16).view(torch_dtype(dtype))[0]
    for bad in (ones, float("inf")):
        run, out = _sequence(T, N, H, dtype, 8901, bad)
        run()
        torch.cuda.synchronize()
        assert torch.isnan(out[0][T, 0]).any()
        assert all(torch.equal(a[:, 1:], b[:, 1:]) for a, b in zip(out, clean))


def test_blocks_that_share_a_sample_in_a_graph():
    """Captured: every replay gives what the eager calls give."""
    run, out = _sequence(5, 50, 256, "f32", 8902)
    run()
    torch.cuda.synchronize()
    want = [o.clone() for o in out]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured = B.gru_seq_blocks(torch.float32, 5, 50, 256)
        run()
    assert captured == B.gru_seq_blocks(torch.float32, 5, 50, 256) == 4
    for _ in range(3):
        for o in (out[0][1:], *out[1:]):
            o.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("H", [64, 256])
def test_gates_at_the_ends_of_their_range(H):
    """Pre-activations from -inf to inf, where exp would overflow, around the seam of tanh's two forms, and NaN: r, z and n against
    torch in 64 bits (the gates' own arithmetic, no products: a zero state).  4 ulp of fp32 next to values of at most one."""
    a = torch.tensor([0.0, -0.0, 1e-30, 1e-4, 0.7499999, 0.75, 0.7500001, 1.0, 8.9, 20.0, 43.9, 44.1, 87.0, 88.5, 104.0, 1e30, float("inf"), float("nan")])
    a = torch.cat([a, -a]).double()
    N = 4
    gi = a[torch.arange(N * 3 * H) % a.numel()].view(1, N, 3 * H).float().cuda()
    zero = lambda *s: torch.zeros(s, device="cuda:0")
    h, saved = zero(2, N, H), zero(1, N, 4 * H)
    B.gru_seq_fwd(gi, zero(3 * H, H), zero(3 * H), zero(3 * H), h, saved)
    torch.cuda.synchronize()
    x, got = gi[0].double().cpu(), saved[0].double().cpu()
    for k, f in enumerate((torch.sigmoid, torch.sigmoid, torch.tanh)):
        # n adds r times a product of zeros to its own argument: NaN where r is
        want, have = f(x[:, k * H:(k + 1) * H] + (0 * torch.sigmoid(x[:, :H]) if k == 2 else 0)), got[:, k * H:(k + 1) * H]
        assert torch.equal(torch.isnan(want), torch.isnan(have))
        assert ((want - have).nan_to_num().abs() <= 2.0 ** -22 * want.nan_to_num().abs() + 2.0 ** -126).all()


# Blocks that share a sample: sequences too short to tell each other their XCD, the shortest that do, and longer ones, against one block a
# sample.  (Forward the same products in the same order; the sums of the backward pass too.)
@pytest.mark.parametrize("dtype,N,H", [("f32", 9, 256), ("f32", 70, 224), ("bf16", 5, 200)])
# The blocks of a sample on one XCD, whose L2 they exchange through, and on several, through memory.
@pytest.mark.parametrize("far", [None, "1"])
@pytest.mark.parametrize("T", [2, 3, 4, 5, 17])
def test_exchange_between_blocks(T, far, N, H, dtype, nsk_env):
    nsk_env("NSK_GRU_FAR", far) if far else None
    dt = torch_dtype(dtype)
    g = torch.Generator(device="cuda").manual_seed(T)
    r = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    gi, w, b_ih, b_hh = r(T, N, 3 * H).to(dt), (r(3 * H, H) / H ** 0.5).to(dt), 0.3 * r(3 * H), 0.3 * r(3 * H)
    h0, dh, wt = r(N, H).to(dt), r(N, H).to(dt), None
    wt = w.t().contiguous()
    got = []
    for split in (None, "1"):
        nsk_env("NSK_GRU_SPLIT", split) if split else None
        h = torch.full((T + 1, N, H), 7.0, device="cuda", dtype=dt)
        h[0] = h0
        saved = torch.full((T, N, 4 * H), 7.0, device="cuda", dtype=dt)
        dgi, dgh, scratch = torch.full((T, N, 3 * H), 7.0, device="cuda", dtype=dt), torch.full((T, N, 3 * H), 7.0, device="cuda", dtype=dt), torch.empty((2, N, H), device="cuda", dtype=dt)
        B.gru_seq_fwd(gi, w, b_ih, b_hh, h, saved)
        B.gru_seq_bwd(saved, h, dh, wt, dgi, dgh, scratch)
        torch.cuda.synchronize()
        got.append((h, saved, dgi, dgh))
    for a, b in zip(*got):
        assert torch.isfinite(a.float()).all()
        assert max_rel_err(host(a), host(b)) <= TOL[dtype]
