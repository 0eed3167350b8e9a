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
