"""The roll-forward of a sequence does not depend on the other sequences of its batch: state and outputs are bit-identical
alone and beside shorter, longer, empty and left-alone sequences, on both sides of the length where its kernel changes (a
batch with both kinds takes two launches).  On the CPU emulator and on the GPU."""
import numpy as np
import pytest
import torch

from test_kernel_emulation import _emulate, emu_binary  # noqa: F401  (the fixture that builds the emulator)
from workloads import LayerShape, make_workload
from workloads.gen import _gen, draw_layer_inputs

SHAPES = {"n128": (2, 32, 128, 1, 64), "n16": (4, 64, 16, 2, 64)}
BATCHES = [[4, 5], [7, 8], [1, 70, 4, 0, 33, 5], [64, 1, 2]]


def _workload(dims, lens, device, io):
    shape = LayerShape(*dims, io)
    wl = make_workload(2, device, seed=43, shape=shape, batch=len(lens), len_range=(1, 2))
    wl.seqlens = list(lens)
    wl.cu_seqlens = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.inputs = draw_layer_inputs(shape, int(sum(lens)), _gen(device, 44), device)
    wl.ckpt_pos = [[n] if n else [] for n in lens]
    H, P, N = dims[:3]
    wl.init_state = [torch.randn((H, P, N), generator=_gen(device, 45 + b), device=device) for b in range(len(lens))]
    return wl


def _alone(wl, b):
    """Sequence b as a batch of its own."""
    import copy
    one = copy.copy(wl)
    lo, hi = int(wl.cu_seqlens[b]), int(wl.cu_seqlens[b + 1])
    one.seqlens, one.cu_seqlens = [hi - lo], np.asarray([0, hi - lo], np.int32)
    one.inputs = type(wl.inputs)(*(t[lo:hi].clone() for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)))
    one.ckpt_pos, one.init_state, one.init_kind = [wl.ckpt_pos[b]], [wl.init_state[b]], [wl.init_kind[b]]
    return one


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("lens", BATCHES)
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_emulated_neighbours(emu_binary, tmp_path, shape, lens, io):  # noqa: F811
    wl = _workload(SHAPES[shape], lens, "cpu", io)
    y, st, _ = _emulate(emu_binary, wl, wl.init_state, tmp_path, 0, "end", advance=True)
    for b, n in enumerate(lens):
        lo, hi = int(wl.cu_seqlens[b]), int(wl.cu_seqlens[b + 1])
        if n == 0:
            assert np.array_equal(st[b], wl.init_state[b].numpy())
            continue
        one = _alone(wl, b)
        sub = tmp_path / f"alone{b}"
        sub.mkdir()
        y1, st1, _ = _emulate(emu_binary, one, one.init_state, sub, 0, "end", advance=True)
        assert np.array_equal(st1[0], st[b]), f"state of sequence {b} ({n} tokens)"
        assert np.array_equal(y1, y[lo:hi]), f"outputs of sequence {b} ({n} tokens)"


def _gpu_advance(wl, state_dtype, skip=()):
    import paper_2411_19379_amd as ssm
    s, inp = wl.shape, wl.inputs
    tdt = {"f32": torch.float32, "f16": torch.float16}[state_dtype]
    states = [v.to(tdt).clone() for v in wl.init_state]
    plan = ssm.Plan(s.nheads, s.headdim, s.d_state, s.ngroups, s.chunk, s.io_dtype, wl.cu_seqlens, None,
                    state_dtype=state_dtype)
    y = torch.full_like(inp.x, 7.0)
    ssm.ssm_state_advance(plan.handle, inp.x.data_ptr(), inp.dt.data_ptr(), wl.A.data_ptr(), inp.B.data_ptr(),
                          inp.C.data_ptr(), wl.D.data_ptr(), [None if b in skip else t.data_ptr() for b, t in enumerate(states)],
                          y.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    plan.close()
    return y, states


@pytest.mark.gpu
@pytest.mark.parametrize("state_dtype", ["f32", "f16"])
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("lens", BATCHES + [[1] * 65 + [40] * 2 + [6]])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_gpu_neighbours(shape, lens, io, state_dtype):
    print(f"roll-forward alone and in a batch: {shape} {lens} {io} {state_dtype}", flush=True)
    wl = _workload(SHAPES[shape], lens, "cuda:0", io)
    skip = (len(lens) - 1,)
    y, st = _gpu_advance(wl, state_dtype, skip)
    for b, n in enumerate(lens):
        lo, hi = int(wl.cu_seqlens[b]), int(wl.cu_seqlens[b + 1])
        if n == 0 or b in skip:
            assert torch.equal(st[b], wl.init_state[b].to(st[b].dtype)) and bool((y[lo:hi] == 7.0).all())
            continue
        y1, st1 = _gpu_advance(_alone(wl, b), state_dtype)
        assert torch.equal(st1[0], st[b]) and torch.equal(y1, y[lo:hi]), f"sequence {b} ({n} tokens)"
