"""The per-call state pointers: null pointers in any form through the binding; and the two ways in which they reach the
kernels, in the launch's own arguments up to 64 sequences and through a device array beyond, at that edge and for every
entry point that takes them.  A sequence's results do not depend on the way: bit-identical in one batch of 64 or 65 and in
two halves."""
import numpy as np
import pytest
import torch

import paper_2411_19379_amd as ssm
from paper_2411_19379_amd import binding
from workloads import LayerShape
from workloads.gen import _gen, draw_layer_inputs, draw_layer_params

DEV = "cuda:0"


@pytest.mark.parametrize("nulls", [[None, None], [0, None], np.zeros(2, np.int64), (False, 0.0)])
def test_null_pointers_in_any_form(nulls):
    plan = ssm.Plan(4, 16, 16, 1, 64, "f32", [0, 3, 5], None)
    assert list(binding._ptr_array(plan.handle, nulls)) == [None, None]
    assert list(binding._ptr_array(plan.handle, [0, 4096])) == [None, 4096]
    plan.close()


def _batch(dims, io, n):
    """n sequences of 16 or 32 tokens (every cut of the batch is 16-byte aligned), two of three from a cached state."""
    H, P, N = dims[:3]
    shape, g = LayerShape(*dims, io), _gen(DEV, 7)
    lens = [16 if b % 2 else 32 for b in range(n)]
    A, D = draw_layer_params(shape, g, DEV)
    inp = draw_layer_inputs(shape, sum(lens), g, DEV)
    states = [None if b % 3 == 2 else torch.randn((H, P, N), generator=g, device=DEV) for b in range(n)]
    return lens, A, D, inp, states


def _cuts(lens, parts):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    edges = [0, len(lens)] if parts == 1 else [0, len(lens) // 2, len(lens)]
    return [(lo, hi, int(cu[lo]), int(cu[hi]), cu[lo:hi + 1] - cu[lo]) for lo, hi in zip(edges, edges[1:])]


SHAPES = {"split": ((4, 64, 16, 2, 64), "bf16"), "f32": ((4, 32, 64, 2, 64), "f32"), "valu": ((4, 24, 40, 2, 64), "f32"),
          "mfma": ((4, 64, 128, 2, 64), "bf16")}


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 65])
@pytest.mark.parametrize("entry", ["ssm_prefill", "ssm_prefill_noalloc"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_gpu_prefill(shape, entry, n):
    print(f"{entry} of {n} sequences, {shape}", flush=True)
    dims, io = SHAPES[shape]
    lens, A, D, inp, states = _batch(dims, io, n)

    def run(parts):
        ys, sts = [], []
        for lo, hi, t0, t1, cu in _cuts(lens, parts):
            plan = ssm.Plan(*dims, io, cu, [[k] for k in lens[lo:hi]])
            y, st = ssm.prefill(plan, inp.x[t0:t1], inp.dt[t0:t1], A, inp.B[t0:t1], inp.C[t0:t1], D, states[lo:hi],
                                entry=getattr(binding, entry))
            torch.cuda.synchronize()
            plan.close()
            ys.append(y), sts.append(st)
        return torch.cat(ys), torch.cat(sts)

    one, two = run(1), run(2)
    assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1]) and bool(torch.isfinite(one[1]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 65])
@pytest.mark.parametrize("shape", ["split", "f32", "mfma"])
def test_gpu_roll_forward(shape, n):
    print(f"roll-forward of {n} sequences, {shape}", flush=True)
    dims, io = SHAPES[shape]
    lens, A, D, inp, states = _batch(dims, io, n)

    def run(parts):
        work, y = [None if s is None else s.clone() for s in states], torch.zeros_like(inp.x)
        for lo, hi, t0, t1, cu in _cuts(lens, parts):
            plan = ssm.Plan(*dims, io, cu, None)
            ssm.ssm_state_advance(plan.handle, inp.x[t0].data_ptr(), inp.dt[t0].data_ptr(), A.data_ptr(),
                                  inp.B[t0].data_ptr(), inp.C[t0].data_ptr(), D.data_ptr(),
                                  [None if s is None else s.data_ptr() for s in work[lo:hi]], y[t0].data_ptr(),
                                  torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            plan.close()
        return work, y

    (s1, y1), (s2, y2) = run(1), run(2)
    assert torch.equal(y1, y2)
    for a, b, s in zip(s1, s2, states):
        assert (a is None and b is None) or (torch.equal(a, b) and not torch.equal(a, s))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 65])
def test_gpu_convolution(n):
    print(f"convolution of {n} sequences", flush=True)
    lens, C, K = [16 if b % 2 else 32 for b in range(n)], 64, 4
    g = torch.Generator(device=DEV).manual_seed(5)
    x, w, bias = (torch.randn(s, generator=g, device=DEV) for s in ((sum(lens), C), (C, K), (C,)))
    cached = [None if b % 3 == 2 else torch.randn((C, K), generator=g, device=DEV) for b in range(n)]

    def run(parts):
        out, sts = torch.zeros_like(x), []
        for lo, hi, t0, t1, cu in _cuts(lens, parts):
            plan = ssm.Plan(4, 16, 16, 1, 64, "f32", cu, [[k] for k in lens[lo:hi]])
            st = torch.zeros((hi - lo, C, K), device=DEV)
            ssm.ssm_conv1d_prefill(plan.handle, C, K, x[t0].data_ptr(), w.data_ptr(), bias.data_ptr(),
                                   [None if s is None else s.data_ptr() for s in cached[lo:hi]], out[t0].data_ptr(),
                                   st.data_ptr(), 1, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            plan.close()
            sts.append(st)
        return out, torch.cat(sts)

    one, two = run(1), run(2)
    assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1])
