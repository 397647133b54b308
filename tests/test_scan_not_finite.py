"""What an infinity or NaN in x, B, C or a cached state becomes in the fp32 and split-operand scans: states and outputs are
infinite or NaN exactly where, and with the sign that, the sums over the tokens of a tile are,
    y_i = e^{l_i} (S C_i) + sum_{j<=i} (C_i.B_j) e^{l_i-l_j} dt_j x_j + D x_i,   S' = e^{l_q} S + sum_j e^{l_q-l_j} dt_j x_j B_j^T
computed here term by term in 64 bits, on whole tiles and on ones with rows past the end.  On the emulator and on the GPU."""
import numpy as np
import pytest
import torch

from helpers import gpu_run, rel_err
from test_kernel_emulation import _emulate, emu_binary  # noqa: F401  (the fixture that builds the emulator)
from test_scan_split import _workload

INF, NAN = float("inf"), float("nan")


def _plain(wl, init, unit):
    """The sums above over units of `unit` tokens of one sequence, and the states at its checkpoints."""
    f = lambda t: t.float().cpu().numpy().astype(np.float64)  # noqa: E731
    x, dt, B, C, A, D = (f(t) for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C, wl.A, wl.D))
    T, H, P = x.shape
    G, N = B.shape[1:]
    S = np.zeros((H, P, N)) if init is None else f(init).copy()
    y, states, pos = np.zeros((T, H, P)), [], 0
    while pos < T:
        stop = min([c for c in wl.ckpt_pos[0] if c > pos] + [T, pos + unit])
        tok = slice(pos, stop)
        with np.errstate(all="ignore"):
            for h in range(H):
                g, ell = h // (H // G), np.cumsum(dt[tok, h] * A[h])
                Sn = np.exp(ell[-1]) * S[h]
                for i in range(stop - pos):
                    acc = np.exp(ell[i]) * sum(S[h][:, n] * C[pos + i, g, n] for n in range(N)) + D[h] * x[pos + i, h]
                    for j in range(i + 1):
                        acc = acc + (C[pos + i, g] @ B[pos + j, g]) * np.exp(ell[i] - ell[j]) * dt[pos + j, h] * x[pos + j, h]
                    y[pos + i, h] = acc
                    Sn = Sn + np.outer(np.exp(ell[-1] - ell[i]) * dt[pos + i, h] * x[pos + i, h], B[pos + i, g])
                S[h] = Sn
        pos = stop
        if pos in wl.ckpt_pos[0]:
            states.append(S.copy())
    return y, np.stack(states)


def _same(got, want, tol):
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    assert not ok.any() or max(rel_err(got[ok], want[ok])) <= tol


# where the value goes: (tensor, token or None, index behind the token)
SPOTS = {"x_first": ("x", 0, (0, 17)), "x_last_of_a_part": ("x", 40, (0, 3)), "B": ("B", 13, (0, 5)),
         "B_last_of_a_part": ("B", 40, (0, 0)), "C": ("C", 20, (0, 7)), "state": ("init", None, (0, 9, 11))}
DIMS = [(1, 32, 16, 1, 64), (1, 48, 64, 1, 64), (1, 48, 128, 1, 16)]


def _spoiled(dims, io, spot, value, device):
    wl = _workload(dims, [41], device, io=io)
    wl.ckpt_pos = [[10, 32, 41]]
    H, P, N = dims[:3]
    init = torch.randn((H, P, N), generator=torch.Generator().manual_seed(3)).to(device)
    name, tok, idx = SPOTS[spot]
    if name == "init":
        init[idx] = value
    else:
        getattr(wl.inputs, name)[(tok, *idx)] = value
    wl.init_state = [init]
    unit = min(dims[4], 16 if io == "f32" else 32)
    return wl, *_plain(wl, init, unit)


@pytest.mark.parametrize("value", [INF, -INF, NAN])
@pytest.mark.parametrize("spot", sorted(SPOTS))
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("dims", DIMS)
def test_emulated(emu_binary, tmp_path, monkeypatch, dims, io, spot, value):  # noqa: F811
    wl, y_ref, st_ref = _spoiled(dims, io, spot, value, "cpu")
    for waves in ("0", "1"):
        monkeypatch.setenv("EMU_F32_WAVES", waves)
        y, st, _ = _emulate(emu_binary, wl, wl.init_state, tmp_path, 0, "end")
        (tmp_path / "out_0_end_None_False_None_False_None.bin").unlink()
        _same(st.astype(np.float64), st_ref, 1e-5)
        _same(y, y_ref, 1e-5 if io == "f32" else 2.0 ** -8 + 1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("value", [INF, -INF, NAN])
@pytest.mark.parametrize("spot", sorted(SPOTS))
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("dims", DIMS)
def test_gpu(dims, io, spot, value):
    print(f"{value} in {spot}, {dims} {io}", flush=True)
    wl, y_ref, st_ref = _spoiled(dims, io, spot, value, "cuda:0")
    y, st, _ = gpu_run(wl, wl.init_state)
    _same(st.cpu().numpy().astype(np.float64), st_ref, 1e-5)
    _same(y.float().cpu().numpy().astype(np.float64), y_ref, 1e-5 if io == "f32" else 2.0 ** -8 + 1e-5)
