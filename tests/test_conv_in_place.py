"""The convolution where a sequence's cached state is updated in place: its initial state is the slot of its only checkpoint.
Few tiles, which the kernel otherwise cuts into parts that run in any order.  On the emulator with the workgroups from the last
to the first, on the GPU against a run with states apart."""
import numpy as np
import pytest
import torch

from test_kernel_emulation import CONV_CASES, emu_conv_binary  # noqa: F401  (the fixture that builds the emulator)
from test_kernel_emulation import test_conv1d_matches_oracle as conv_case

LENS = [64, 9, 33, 17, 1]


@pytest.mark.parametrize("K", [1, 4])
@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_emulated(emu_conv_binary, tmp_path, monkeypatch, io, K):  # noqa: F811
    CONV_CASES["in_place"] = ((4, 16, 16, 1, 64) if io == "f32" else (2, 64, 128, 1, 64),
                              [16, 9, 13] if io == "f32" else LENS[:3], [[16], [9], [13]] if io == "f32" else [[64], [9], [33]])
    monkeypatch.setenv("EMU_LAST_BLOCK_FIRST", "1")
    monkeypatch.setenv("EMU_IN_PLACE", "1")
    conv_case(emu_conv_binary, tmp_path, io, "in_place", K)


@pytest.mark.gpu
@pytest.mark.parametrize("K", [1, 4])
def test_gpu(K):
    import paper_2411_19379_amd as ssm

    C, T, dev = 5376, sum(LENS), "cuda:0"
    g = torch.Generator(device=dev).manual_seed(K)
    draw = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    x, w, bias = draw(T, C).bfloat16(), draw(C, K), draw(C)
    cached = draw(len(LENS), C, K).bfloat16()
    plan = ssm.Plan(80, 64, 128, 1, 256, "bf16", np.concatenate([[0], np.cumsum(LENS)]), [[n] for n in LENS])
    stream = torch.cuda.current_stream().cuda_stream

    def run(states, out_states):
        out = torch.empty_like(x)
        ssm.ssm_conv1d_prefill(plan.handle, C, K, x.data_ptr(), w.data_ptr(), bias.data_ptr(),
                               [states[b].data_ptr() for b in range(len(LENS))], out.data_ptr(), out_states.data_ptr(), 1, stream)
        torch.cuda.synchronize()
        return out

    apart = torch.empty_like(cached)
    want = run(cached, apart)
    for rep in range(20):
        print(f"in place, K={K}, pass {rep}", flush=True)
        states = cached.clone()
        got = run(states, states)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
        assert torch.equal(states.view(torch.int16), apart.view(torch.int16))
    plan.close()
