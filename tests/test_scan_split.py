"""The split-operand scan (bf16 storage, fp32 results) at the edges of its dispatch: every block count of d_state, heads of
one to eight 16-channel slices, units of 32 tokens with every kind of remainder, tiles of 16 and 32 tokens, and the same kernel as
the roll-forward; on the CPU emulator (wave orders, bounds, unwritten outputs) and on the GPU.  Every product is exact and
added up in fp32 as in the fp32 kernel, so the bounds are the fp32 ones: 1e-5, and 2^-8 of the value where y is rounded to
bf16.  Then what a token whose x is not finite may reach: its own channel, from its own position on."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2411_19379_amd.binding import load_library
from helpers import gpu_run, oracle_on_heads, rel_err
from test_kernel_emulation import _emulate, _oracle, emu_binary  # noqa: F401  (the fixture that builds the emulator)
from workloads import LayerShape, make_workload
from workloads.gen import _gen, draw_layer_inputs

Y_TOL = 2.0 ** -8 + 1e-5


def _workload(dims, lens, device, seed=41, io="bf16"):
    H, P, N, G, chunk = dims
    shape = LayerShape(H, P, N, G, chunk, io)
    wl = make_workload(2, device, seed=seed, shape=shape, batch=len(lens), len_range=(1, 2))
    wl.seqlens = list(lens)
    wl.cu_seqlens = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.inputs = draw_layer_inputs(shape, int(sum(lens)), _gen(device, seed + 1), device)
    rs = np.random.RandomState(seed)
    wl.ckpt_pos = [sorted({int(v) for v in rs.randint(1, n + 1, size=2)} | {n}) if n else [] for n in lens]
    return wl


EMU_CASES = {
    "n16_four_slices": ((1, 64, 16, 1, 64), [70, 1]),
    "n16_one_slice_tiles_of_16": ((2, 48, 16, 2, 16), [33, 0, 65]),
    "n32": ((3, 32, 32, 1, 64), [32, 31]),
    "n64": ((2, 32, 64, 2, 64), [63, 96]),
}


@pytest.mark.parametrize("case", sorted(EMU_CASES))
def test_emulated_scan(emu_binary, tmp_path, case):  # noqa: F811
    wl = _workload(*EMU_CASES[case], "cpu")
    init = list(wl.init_state)
    y_ref, st_ref = _oracle(wl, init)
    first = None
    for order, align in ((0, "end"), (1, "start"), (2, "end")):
        y, st, raw = _emulate(emu_binary, wl, init, tmp_path, order, align)
        assert np.isfinite(y).all() and np.isfinite(st).all()
        assert max(rel_err(y, y_ref)) <= Y_TOL
        assert max(rel_err(st, st_ref)) <= 1e-5
        first = raw if first is None else first
        assert np.array_equal(first, raw)


def test_emulated_roll_forward(emu_binary, tmp_path):  # noqa: F811
    wl = _workload((2, 32, 128, 1, 64), [33, 5, 0], "cpu")
    wl.ckpt_pos = [[n] if n else [] for n in wl.seqlens]
    init = list(wl.init_state)
    y_ref, st_ref = _oracle(wl, init)
    for order, align in ((0, "end"), (1, "start")):
        y, st, _ = _emulate(emu_binary, wl, init, tmp_path, order, align, advance=True)
        assert max(rel_err(y, y_ref)) <= Y_TOL
        assert max(rel_err(st[:2], st_ref)) <= 1e-5


def _spoil(x, tok, h, p, value):
    x[tok, h, p] = value


def _check_reach(y, y0, st, st0, ckpts, tok, h, p):
    """Sequence 0 only: y [T,H,P] and states in checkpoint order, with and without the spoiled value."""
    assert np.isfinite(y0).all() and np.isfinite(st0).all()
    other = np.ones(y.shape, bool)
    other[:, h, p] = False
    assert np.array_equal(y[other], y0[other])
    assert np.array_equal(y[:tok, h, p], y0[:tok, h, p])
    assert not np.isfinite(y[tok, h, p])
    for k, c in enumerate(ckpts):
        keep = np.ones(st0[k].shape, bool)
        if c > tok:
            keep[h, p] = False
            assert not np.isfinite(st[k][h, p]).all()
        assert np.array_equal(st[k][keep], st0[k][keep])


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("tok", [0, 13, 21, 40])
def test_emulated_value_that_is_not_finite(emu_binary, tmp_path, tok, io, value):  # noqa: F811
    dims, lens = ((1, 32, 16, 1, 64), [41])
    wl = _workload(dims, lens, "cpu", io=io)
    wl.ckpt_pos = [[10, 32, 41]]
    init = list(wl.init_state)
    y0, st0, _ = _emulate(emu_binary, wl, init, tmp_path, 0, "end")
    _spoil(wl.inputs.x, tok, 0, 17, value)
    sub = tmp_path / "spoiled"
    sub.mkdir()
    y, st, _ = _emulate(emu_binary, wl, init, sub, 0, "end")
    _check_reach(y, y0, st, st0, wl.ckpt_pos[0], tok, 0, 17)


GPU_CASES = dict(EMU_CASES)
GPU_CASES.update({
    "n16_many": ((64, 64, 16, 1, 256), [260, 64, 17, 3, 128]),
    "n32_four_slices": ((40, 128, 32, 4, 256), [90, 250]),
    "n64_two_slices_shared": ((150, 64, 64, 1, 256), [33, 180]),
    "n64_eight_waves": ((2, 64, 64, 1, 256), [300]),
    "odd_slices": ((5, 80, 32, 5, 32), [95, 32]),
    "n16_packed": ((32, 64, 16, 1, 256), [300, 64, 17, 128, 33, 250, 90, 512]),
    "n16_two_slices": ((64, 32, 16, 1, 256), [100, 33, 40, 70]),
})
GPU_SLICES = {"n16_packed": 4, "n16_two_slices": 2, "n32_four_slices": 4, "n64_two_slices_shared": 2, "n16_many": 2}


@pytest.mark.gpu
@pytest.mark.parametrize("case", sorted(GPU_CASES))
def test_gpu_scan(case):
    print(f"split-operand scan {case}", flush=True)
    wl = _workload(*GPU_CASES[case], "cuda:0")
    init = [None if s is None else s.cpu().numpy() for s in wl.init_state]
    y, st, info = gpu_run(wl, wl.init_state)
    assert info.path == 0
    if case in GPU_SLICES:  # several slices per workgroup
        (H, P, N, _, _), lens = GPU_CASES[case]
        assert load_library().ssm_f32_slices(1, N, P, ctypes.c_int64(len(lens) * H)) == GPU_SLICES[case]
    y_ref, st_ref = oracle_on_heads(wl, None, init)
    assert max(rel_err(y.float().cpu().numpy(), y_ref)) <= Y_TOL
    for k in range(st_ref.shape[0]):
        assert max(rel_err(st[k].cpu().numpy(), st_ref[k])) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("state_dtype,tdt,tol", [("f32", torch.float32, 1e-5), ("f16", torch.float16, 2.0 ** -11 + 1e-5),
                                                 ("bf16", torch.bfloat16, 2.0 ** -8 + 1e-5)])
@pytest.mark.parametrize("H,lens", [(3, [6, 31, 33]), (96, [65, 256, 160])])
def test_gpu_roll_forward(H, lens, state_dtype, tdt, tol):
    import paper_2411_19379_amd as ssm
    print(f"roll-forward {lens} H={H} {state_dtype}", flush=True)
    P, N, G = 48, 128, 3
    wl = _workload((H, P, N, G, 64), lens, "cuda:0")
    inp = wl.inputs
    g = torch.Generator(device="cuda:0").manual_seed(3)
    states = [torch.randn((H, P, N), generator=g, device="cuda:0").to(tdt) for _ in lens]
    before = [s.float().cpu().numpy() for s in states]
    plan = ssm.Plan(H, P, N, G, 64, "bf16", wl.cu_seqlens, None, state_dtype=state_dtype)
    y = torch.full_like(inp.x, float("nan"))
    ssm.ssm_state_advance(plan.handle, inp.x.data_ptr(), inp.dt.data_ptr(), wl.A.data_ptr(), inp.B.data_ptr(),
                          inp.C.data_ptr(), wl.D.data_ptr(), [s.data_ptr() for s in states], y.data_ptr(),
                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    plan.close()
    wl.ckpt_pos = [[n] for n in lens]
    y_ref, st_ref = oracle_on_heads(wl, None, before)
    assert max(rel_err(y.float().cpu().numpy(), y_ref)) <= Y_TOL
    for b in range(len(lens)):
        assert max(rel_err(states[b].float().cpu().numpy(), st_ref[b])) <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("tok", [0, 18, 63, 69])
def test_gpu_value_that_is_not_finite(tok, io):
    print(f"x not finite at token {tok}, {io}", flush=True)
    wl = _workload((4, 64, 16, 2, 64), [70], "cuda:0", io=io)
    wl.ckpt_pos = [[10, 32, 70]]
    y0, st0, _ = gpu_run(wl, wl.init_state)
    _spoil(wl.inputs.x, tok, 2, 37, float("inf"))
    y, st, _ = gpu_run(wl, wl.init_state)
    _check_reach(y.float().cpu().numpy(), y0.float().cpu().numpy(), st.cpu().numpy(), st0.cpu().numpy(), wl.ckpt_pos[0],
                 tok, 2, 37)
