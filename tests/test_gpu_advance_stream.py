"""Decode steps whose states are large enough to pass by the caches: bit-identical to the same sequences in batches below
that limit, in every storage type of the states, with a sequence left alone in between."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("state_dtype,tdt,batch", [("f32", torch.float32, 34), ("f16", torch.float16, 66),
                                                   ("bf16", torch.bfloat16, 66), ("f32", torch.float32, 33),
                                                   ("f32", torch.float32, 65), ("f16", torch.float16, 137),
                                                   ("f16", torch.float16, 138)])
def test_large_batches_equal_small_ones(state_dtype, tdt, batch):
    import paper_2411_19379_amd as ssm
    print(f"decode of {batch} sequences in one call and in thirds, {state_dtype}", flush=True)
    H, P, N, G = 128, 64, 128, 8
    g = torch.Generator(device=DEV).manual_seed(11)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV)

    x, B, C = (normal(batch, *s).bfloat16() for s in ((H, P), (G, N), (G, N)))
    dt = (0.1 * torch.rand((batch, H), generator=g, device=DEV)).bfloat16()
    A, D = -1.0 - normal(H).abs(), normal(H)
    states = normal(batch, H, P, N).to(tdt)
    assert states.numel() * states.element_size() > 128 << 20
    skipped = batch // 2

    def step(lo, hi, st, y):
        plan = ssm.Plan(H, P, N, G, 256, "bf16", np.arange(hi - lo + 1, dtype=np.int32), None, state_dtype=state_dtype)
        ptrs = [None if b == skipped else st[b].data_ptr() for b in range(lo, hi)]
        ssm.ssm_state_advance(plan.handle, x[lo].data_ptr(), dt[lo].data_ptr(), A.data_ptr(), B[lo].data_ptr(),
                              C[lo].data_ptr(), D.data_ptr(), ptrs, y[lo].data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        plan.close()

    one, y_one = states.clone(), torch.zeros_like(x)
    step(0, batch, one, y_one)
    parts, y_parts = states.clone(), torch.zeros_like(x)
    edges = [0, batch // 3, 2 * batch // 3, batch]
    for lo, hi in zip(edges, edges[1:]):
        step(lo, hi, parts, y_parts)
    assert torch.equal(one, parts) and torch.equal(y_one, y_parts)
    assert torch.equal(one[skipped], states[skipped]) and not torch.equal(one[0], states[0])
