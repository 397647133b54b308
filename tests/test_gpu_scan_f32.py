"""The fp32 matrix-core scan at the edges of its dispatch: every block count of d_state, one to four 16-channel slices per
workgroup (few and many streams), tiles of every remainder, more tiles than waves, and the same kernel as the roll-forward
on both sides of its threshold.  Against the fp64 oracle; fp32 sums of at most 16 + d_state terms per output and one
rounding per tile in the state: 1e-5 (and 2^-8 of the value where y is stored in bf16)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2411_19379_amd as ssm
from helpers import gpu_run, oracle_on_heads, rel_err
from workloads import LayerShape, make_workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# H, P, N, G, io; sequence lengths
CASES = {
    "n16_one_slice": ((4, 16, 16, 2, "f32"), [1, 15, 16, 17, 300]),
    "n16_two_slices": ((64, 32, 16, 4, "f32"), [33, 90, 160, 1]),
    "n16_four_slices": ((64, 64, 16, 1, "f32"), [70, 260, 5, 64, 17, 3, 40, 8]),
    "n32_three_slices_left_apart": ((6, 48, 32, 3, "f32"), [40, 0, 129]),
    "n32_two_slices": ((64, 32, 32, 2, "f32"), [40, 90, 129, 1]),
    "n32_four_slices": ((64, 64, 32, 2, "f32"), [40, 90, 129, 1]),
    "n64": ((3, 128, 64, 1, "f32"), [140, 1]),
    "n64_two_slices": ((64, 64, 64, 1, "f32"), [140, 1, 33, 50]),
    "n128_one_slice": ((2, 16, 128, 1, "f32"), [16, 129, 260]),
    "n128_two_slices": ((64, 64, 128, 4, "f32"), [31, 150, 64, 9]),
}
SLICES = {"n16_two_slices": 2, "n16_four_slices": 4, "n32_two_slices": 2, "n32_four_slices": 4, "n64_two_slices": 2,
          "n128_two_slices": 2}


@pytest.mark.parametrize("case", sorted(CASES))
def test_fp32_matrix_core_scan(case):
    (H, P, N, G, io), lens = CASES[case]
    print(f"fp32 scan {case}", flush=True)
    wl = make_workload(2, DEV, seed=31, batch=len(lens), len_range=(max(lens), max(lens)), shape=LayerShape(H, P, N, G, 64, io))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    inp = type(wl.inputs)(*(t[:T].contiguous() for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)))
    rs = np.random.RandomState(5)
    ck = [sorted({int(v) for v in rs.randint(1, n + 1, size=2)} | {n}) if n else [] for n in lens]
    init = [None if s is None else s.cpu().numpy() for s in wl.init_state]
    y, st, info = gpu_run(wl, wl.init_state, inputs=inp, cu=cu, ckpt_pos=ck)
    assert info.path == 0
    streams = sum(n > 0 for n in lens) * H
    assert ssm.load_library().ssm_f32_slices(0, N, P, ctypes.c_int64(streams)) == SLICES.get(case, 1)
    y_ref, st_ref = oracle_on_heads(wl, None, init, inputs=inp, cu=cu, ckpt_pos=ck)
    assert max(rel_err(y.float().cpu().numpy(), y_ref)) <= (1e-5 if io == "f32" else 2.0 ** -8 + 1e-5)
    for k in range(st_ref.shape[0]):
        assert max(rel_err(st[k].cpu().numpy(), st_ref[k])) <= 1e-5


@pytest.mark.parametrize("H", [2, 96])
@pytest.mark.parametrize("lens", [[4, 1], [5, 0, 2], [16, 17, 31], [200, 1]])
def test_roll_forward_on_both_sides_of_the_threshold(lens, H):
    print(f"roll-forward {lens} H={H}", flush=True)
    P, N, G = 64, 128, 2
    wl = make_workload(2, DEV, seed=37, batch=len(lens), len_range=(max(lens), max(lens)),
                       shape=LayerShape(H, P, N, G, 64, "bf16"))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    x, dt, B, C = (t[:T].contiguous() for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C))
    g = torch.Generator(device=DEV).manual_seed(3)
    states = [torch.randn((H, P, N), generator=g, device=DEV) for _ in lens]
    before = [s.cpu().numpy().copy() for s in states]
    plan = ssm.Plan(H, P, N, G, 64, "bf16", cu, None)
    for want_y in (False, True):  # without outputs first: the states must come out the same
        work = [s.clone() for s in states]
        y = torch.full_like(x, float("nan")) if want_y else None
        ssm.ssm_state_advance(plan.handle, x.data_ptr(), dt.data_ptr(), wl.A.data_ptr(), B.data_ptr(), C.data_ptr(),
                              wl.D.data_ptr(), [s.data_ptr() for s in work], y.data_ptr() if want_y else None,
                              torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        if not want_y:
            first = work
    plan.close()
    from oracle import ssm_prefill_oracle
    y_ref, st_ref = ssm_prefill_oracle(x.cpu(), dt.cpu(), wl.A.cpu(), B.cpu(), C.cpu(), wl.D.cpu(), cu, before,
                                       [[n] if n else [] for n in lens])
    assert max(rel_err(y.float().cpu().numpy(), y_ref)) <= 2.0 ** -8 + 1e-5
    k = 0
    for b, n in enumerate(lens):
        assert torch.equal(first[b], work[b])
        if n:
            assert max(rel_err(work[b].cpu().numpy(), st_ref[k])) <= 1e-5
            k += 1
        else:
            assert torch.equal(work[b], states[b])
