"""The fp32 and split-operand scans with every number of waves per workgroup that their launch rule can pick (few where the
launch fills the GPU with short sequences; one wave alone keeps the state in its registers) and every number of 16-channel
slices, and the roll-forward through the same kernels: on the emulator with both numbers fixed, on the GPU with batches that
the rules send there.  Against the oracle with the bounds of the other tests of these kernels, and bit-identical whatever
the numbers."""
import numpy as np
import pytest
import torch

from helpers import gpu_run, oracle_on_heads, rel_err
from test_kernel_emulation import _emulate, _oracle, emu_binary  # noqa: F401  (the fixture that builds the emulator)
from test_scan_split import _workload

Y_TOL = {"bf16": 2.0 ** -8 + 1e-5, "f32": 1e-5}

CASES = {
    "n16": ((2, 64, 16, 1, 64), [70, 1, 0, 33]),
    "n32": ((2, 32, 32, 2, 16), [17, 40]),
    "n32_wide": ((1, 64, 32, 1, 64), [33, 3]),
    "n64": ((1, 48, 64, 1, 64), [65, 5]),
    "n64_wide": ((1, 64, 64, 1, 64), [17, 35]),
    "n128_wide": ((1, 32, 128, 1, 64), [19]),
    "n128": ((1, 48, 128, 1, 64), [20, 49]),  # headdim 48: bf16 storage takes the split kernel at d_state 128 too
}


@pytest.mark.parametrize("waves,slices,advance", [(1, 0, False), (2, 0, False), (0, 2, False), (1, 2, False), (8, 4, False),
                                                  (1, 4, False), (1, 0, True), (2, 2, True)])
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_emulated_waves(emu_binary, tmp_path, monkeypatch, case, io, advance, waves, slices):  # noqa: F811
    dims, lens = CASES[case]
    if slices and (dims[1] // 16 % slices or slices > (4 if dims[2] <= 32 else 1 if (io, dims[2]) == ("bf16", 128) else 2)):
        pytest.skip("no such kernel")
    if io == "bf16" and dims[1:3] == (32, 128) and not advance:
        pytest.skip("not these kernels' shape")
    wl = _workload(dims, lens, "cpu", io=io)
    if advance:
        wl.ckpt_pos = [[n] if n else [] for n in lens]
    init = list(wl.init_state)
    y_ref, st_ref = _oracle(wl, init)
    _, _, want = _emulate(emu_binary, wl, init, tmp_path, 0, "end", advance=advance)
    sub = tmp_path / "waves"
    sub.mkdir()
    monkeypatch.setenv("EMU_F32_WAVES", str(waves))
    monkeypatch.setenv("EMU_F32_SLICES", str(slices))
    for order, align in ((0, "end"), (1, "start")):
        y, st, raw = _emulate(emu_binary, wl, init, sub, order, align, advance=advance)
        assert np.array_equal(raw, want)
        assert max(rel_err(y, y_ref)) <= Y_TOL[io]
        if advance:
            st = st[[b for b, n in enumerate(lens) if n]]
        assert max(rel_err(st, st_ref)) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("dims,lens", [
    ((32, 64, 16, 1, 256), [1, 2, 5, 0] * 20),              # more workgroups than four per compute unit, one unit each
    ((64, 32, 32, 2, 256), [30, 33, 70] * 12),
    ((32, 64, 64, 1, 256), [3] * 40 + [100]),               # one long sequence among short ones
    ((24, 48, 128, 1, 64), [9, 20, 16] * 10),
])
def test_gpu_many_short_sequences(dims, lens, io):
    print(f"{len(lens)} short sequences, {dims} {io}", flush=True)
    wl = _workload(dims, lens, "cuda:0", io=io)
    y, st, info = gpu_run(wl, wl.init_state)
    assert info.path == 0
    y_ref, st_ref = oracle_on_heads(wl, None, [None if s is None else s.cpu().numpy() for s in wl.init_state])
    assert max(rel_err(y.float().cpu().numpy(), y_ref)) <= Y_TOL[io]
    for k in range(st_ref.shape[0]):
        assert max(rel_err(st[k].cpu().numpy(), st_ref[k])) <= 1e-5
    # the same sequences in a batch of their own take other numbers of waves: same bits
    few = _workload(dims, lens, "cuda:0", io=io)
    n = 3
    few.seqlens, few.cu_seqlens = lens[:n], wl.cu_seqlens[:n + 1]
    T = int(few.cu_seqlens[-1])
    few.inputs = type(wl.inputs)(*(t[:T].contiguous() for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)))
    few.ckpt_pos = wl.ckpt_pos[:n]
    y1, st1, _ = gpu_run(few, wl.init_state[:n])
    assert torch.equal(y1, y[:T]) and torch.equal(st1, st[:st1.shape[0]])


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_gpu_more_threads_than_a_launch_takes(io):
    """One long sequence among 65535 empty ones at 128 heads: with its waves for every sequence, 2^32 threads and more."""
    print(f"65536 sequences, {io}", flush=True)
    lens = [0] * 65536
    lens[40000] = 2100
    wl = _workload((128, 16, 16, 1, 64), lens[40000:40001], "cuda:0", io=io)
    wl.ckpt_pos = [[2100]]
    y1, st1, _ = gpu_run(wl, wl.init_state[:1])
    wl.seqlens, wl.cu_seqlens = lens, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.ckpt_pos = [[n] if n else [] for n in lens]
    init = [None] * len(lens)
    init[40000] = wl.init_state[0]
    y, st, info = gpu_run(wl, init)
    assert info.path == 0 and torch.equal(y, y1) and torch.equal(st, st1)
