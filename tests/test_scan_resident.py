"""The matrix-core scan with resident states (`scan_resident.hip`): on the CPU emulator against the oracle at the edges of
its tiles, pieces and channel blocks, in any wave order and with guarded buffers; on the GPU where the plan takes it."""
import os
import subprocess

import numpy as np
import pytest
import torch

from helpers import TOL, rel_err
from test_kernel_emulation import (CLANG, CSRC, EMU, ROOT, _convert, _emulate, _oracle, _with_empty_sequence,
                                   emu_binary)  # noqa: F401  (the fixture that builds the other scans)
from workloads import LayerShape, make_workload

# name: (H, P, N, G, chunk), configuration of the generator, its overrides; every group is a multiple of 256 channels
CASES = {
    "ragged": ((4, 64, 128, 1, 64), 2, dict(batch=3, len_range=(1, 300))),
    "long": ((4, 64, 128, 1, 64), 4, dict(seqlen=450, ckpt_every=100)),
    "tiny": ((8, 64, 128, 2, 64), 2, dict(batch=2, len_range=(1, 3))),
    "two_groups": ((8, 64, 128, 2, 32), 2, dict(batch=2, len_range=(20, 120))),
    "p128": ((4, 128, 128, 2, 16), 4, dict(seqlen=130, ckpt_every=64)),
    "empty_seq": ((4, 64, 128, 1, 64), 2, dict(batch=3, len_range=(30, 200))),
    # decay up to 400 times the usual: the masks' exact branch, and pieces that nothing in front of them reaches
    "strong_decay": ((4, 64, 128, 1, 64), 2, dict(batch=2, len_range=(60, 200), a_scale=[1.0, 40.0, 400.0, 0.01])),
    # a hundredth of it: everything in front of a piece reaches all of it
    "p256": ((2, 256, 128, 1, 64), 2, dict(batch=2, len_range=(60, 200))),
    "slow_decay": ((4, 64, 128, 1, 64), 2, dict(batch=2, len_range=(300, 400), a_scale=[0.01, 0.01, 0.02, 0.03])),
}


@pytest.fixture(scope="session")
def emu_resident(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ with bf16 vector support found")
    d = str(tmp_path_factory.mktemp("emu_resident"))
    srcs = [os.path.join(CSRC, "plan.cpp"), os.path.join(EMU, "emu_rt.cpp"), os.path.join(EMU, "emu_main.cpp")]
    for name in ("scan_resident", "scan_valu", "state_advance"):
        _convert(os.path.join(CSRC, name + ".hip"), os.path.join(d, name + ".cpp"))
        srcs.append(os.path.join(d, name + ".cpp"))
    flags = ["-std=c++17", "-O2", "-fno-strict-aliasing", "-ffp-contract=off", "-Wno-psabi", "-Wno-unused-value",
             "-DEMU_RESIDENT", "-I", EMU, "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = [os.path.join(d, os.path.basename(s) + ".o") for s in srcs]
    procs = [subprocess.Popen([CLANG, *flags, "-c", s, "-o", o], stderr=subprocess.PIPE, text=True)
             for s, o in zip(srcs, objs)]
    for p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, err[-3000:]
    out = os.path.join(d, "emu_main")
    subprocess.run([CLANG, *objs, "-o", out], check=True)
    return out


@pytest.mark.parametrize("most,segment", [(None, None), (1, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("case", sorted(CASES))
def test_emulated_scan_matches_oracle(emu_resident, tmp_path, monkeypatch, case, most, segment):
    """`most`, `segment`: tiles per piece and per segment.  Tolerances as for the other matrix-core scan."""
    dims, cfg, kw = CASES[case]
    kw = dict(kw)
    a_scale = kw.pop("a_scale", None)
    wl = make_workload(cfg, "cpu", seed=11, shape=LayerShape(*dims, "bf16"), **kw)
    if a_scale is not None:
        wl.A = wl.A * torch.tensor(a_scale, dtype=wl.A.dtype)
    if case == "empty_seq":
        wl = _with_empty_sequence(wl)
    init = list(wl.init_state)
    y_ref, st_ref = _oracle(wl, init)
    if most:
        monkeypatch.setenv("EMU_PIECES", str(most))
        monkeypatch.setenv("EMU_SEGMENTS", str(segment))
    first = None
    for order, align in ((0, "end"), (1, "start"), (7, "end")):
        y, st, raw = _emulate(emu_resident, wl, init, tmp_path, order, align)
        assert np.all(np.isfinite(y)) and np.all(np.isfinite(st))
        assert max(rel_err(y, y_ref)) <= TOL["bf16"]
        assert max(rel_err(st.astype(np.float64), st_ref)) <= TOL["bf16"]
        first = raw if first is None else first
        assert np.array_equal(first, raw), f"wave order {order} changes the result: LDS race"


@pytest.mark.parametrize("a_scale", [(0.01, 0.01, 0.01, 0.01), (0.01, 400.0, 3.0, 30.0)])
def test_emulated_sums_of_segments(emu_resident, tmp_path, monkeypatch, a_scale):
    """Pieces with up to 40 segments of 16 tokens in front of them, of which groups of eight are summed up for the pieces far
    behind: groups that are needed, that hold two sequences, and that strong decay leaves out."""
    total = sum(lens := [200, 650, 300])
    wl = make_workload(2, "cpu", seed=43, batch=1, len_range=(total, total), shape=LayerShape(4, 64, 128, 1, 16, "bf16"))
    wl.seqlens, wl.cu_seqlens = lens, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.ckpt_pos = [[100, 200], [648], []]
    wl.A = wl.A * torch.tensor(a_scale)
    init = [torch.randn((4, 64, 128), generator=torch.Generator().manual_seed(k)) for k in range(3)]
    y_ref, st_ref = _oracle(wl, init)
    monkeypatch.setenv("EMU_PIECES", "1")
    monkeypatch.setenv("EMU_SEGMENTS", "1")
    for order, align in ((0, "end"), (7, "start")):
        y, st, _ = _emulate(emu_resident, wl, init, tmp_path, order, align)
        assert max(rel_err(y, y_ref)) <= TOL["bf16"]
        assert max(rel_err(st.astype(np.float64), st_ref)) <= TOL["bf16"]


@pytest.mark.parametrize("a_scale", [0.002, 1.0])
def test_emulated_segments_longer_than_the_windows_looked_back_over(emu_resident, tmp_path, monkeypatch, a_scale):
    """A piece of 18 tiles that another continues: its segment looks back over more than 1024 tokens, or stops before."""
    wl = make_workload(4, "cpu", seed=47, shape=LayerShape(4, 64, 128, 1, 64, "bf16"), seqlen=2300, ckpt_every=1150)
    wl.A = wl.A * a_scale
    init = [torch.randn((4, 64, 128), generator=torch.Generator().manual_seed(3))]
    y_ref, st_ref = _oracle(wl, init)
    monkeypatch.setenv("EMU_PIECES", "19")
    y, st, _ = _emulate(emu_resident, wl, init, tmp_path, 0, "end")
    assert max(rel_err(y, y_ref)) <= TOL["bf16"]
    assert max(rel_err(st.astype(np.float64), st_ref)) <= TOL["bf16"]


# What is not finite in an input, or becomes so in fp16, must reach what it reaches in the other matrix-core scan and nothing
# more.  One sequence of 150 tokens; heads of the usual decay, of one whose tiles leave the range of the masks' factors and of
# ones in between (16 with steps of 0.1 is the end of the usual ranges).
# The tiles are those of tokens 0, 64, 70 and 134 on, the second and the fourth partial.
SPOILED = ["state_above_fp16", "C_infinite", "C_infinite_steps_of_0.1", "B_infinite_in_a_partial_tile", "B_above_fp16_in_a_partial_tile",
           "step_NaN", "step_infinite", "late_step_NaN"]


def _spoiled(what, device, copies=1):
    """The workload with `copies` equal sequences and their initial states."""
    wl = make_workload(2, "cpu", seed=19, shape=LayerShape(4, 64, 128, 1, 64, "bf16"), batch=1, len_range=(150, 150))
    wl.A = wl.A * torch.tensor([1.0, 40.0, 400.0, 3.0])
    init = torch.randn((4, 64, 128), generator=torch.Generator().manual_seed(5))
    if what == "state_above_fp16":
        init[:, :, 9] = 7e4
    if what.startswith("C_infinite"):
        wl.inputs.C[20, 0, 7] = float("inf")
    if what.startswith("B_"):
        wl.inputs.B[[69, 149], 0, 7] = float("inf") if "infinite" in what else 1e5
        wl.A = wl.A[:1].repeat(4) * torch.tensor([1.0, 2.0, 0.5, 1.0])
    if "step_" in what:
        wl.inputs.dt[110 if "late" in what else 9, 1:] = float(what.split("_")[-1].replace("infinite", "inf"))
    if what.endswith("steps_of_0.1"):
        wl.A = torch.full_like(wl.A, -16.0)
        wl.inputs.dt.fill_(0.1)
    wl.inputs = type(wl.inputs)(*[torch.cat([t] * copies).to(device) for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)])
    wl.A, wl.D = wl.A.to(device), wl.D.to(device)
    wl.seqlens, wl.ckpt_pos = [150] * copies, [[70, 150]] * copies
    wl.cu_seqlens = np.arange(copies + 1, dtype=np.int32) * 150
    return wl, [init.to(device)] * copies


def _same_reach(got, want, tol):
    """Infinite and NaN at the same places; elsewhere the same within `tol` of the value or the rms."""
    assert np.array_equal(np.isnan(got), np.isnan(want)), (np.isnan(got).sum(), np.isnan(want).sum())
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    assert max(rel_err(got[ok], want[ok])) <= tol


@pytest.mark.parametrize("what", SPOILED)
def test_emulated_values_that_are_not_finite(emu_resident, emu_binary, tmp_path, monkeypatch, what):  # noqa: F811
    wl, init = _spoiled(what, "cpu")
    y_ref, st_ref, _ = _emulate(emu_binary, wl, init, tmp_path, 0, "end")
    y, st, _ = _emulate(emu_resident, wl, init, tmp_path, 0, "end")
    assert not np.isfinite(y_ref).all() and np.isfinite(st_ref).all() == (what[0] in "Cs" and "step_" not in what)
    _same_reach(st.astype(np.float64), st_ref.astype(np.float64), 1e-3)  # both round the weighted x to fp16 alike
    _same_reach(y, y_ref, TOL["bf16"])
    if what[0] == "B":  # through the segments too
        monkeypatch.setenv("EMU_PIECES", "2")
        y, st, _ = _emulate(emu_resident, wl, init, tmp_path, 0, "end")
        _same_reach(st.astype(np.float64), st_ref.astype(np.float64), 1e-3)
        _same_reach(y, y_ref, TOL["bf16"])


# An infinity or NaN in a state stays there to the end of the sequence, also in pieces that start without what has decayed: as
# in a sequence that is walked in one go.  (Infinite or NaN is not compared: what is infinite becomes NaN in a tile whose decay
# is zero in fp32.)
STICKY = {"x": ("x", 5, (1, 17)), "B": ("B", 130, (0, 5)), "dt": ("dt", 3, (2,)), "state": ("init", None, (1, 9, 11))}


def _sticky(spot, value, device, tokens, decay):
    wl = make_workload(2, "cpu", seed=29, shape=LayerShape(4, 64, 128, 1, 64, "bf16"), batch=1, len_range=(tokens, tokens))
    wl.A = wl.A * torch.tensor(decay)
    wl.ckpt_pos = [[tokens // 8, tokens // 2, tokens - 1]]
    init = torch.randn((4, 64, 128), generator=torch.Generator().manual_seed(7))
    name, tok, idx = STICKY[spot]
    (init if name == "init" else getattr(wl.inputs, name))[idx if tok is None else (tok, *idx)] = value
    wl.inputs = type(wl.inputs)(*[t.to(device) for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)])
    wl.A, wl.D = wl.A.to(device), wl.D.to(device)
    return wl, [init.to(device)]


def _same_finite(got, want, tol):
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok), ((~np.isfinite(got)).sum(), (~ok).sum())
    assert not ok.all() and max(rel_err(got[ok], want[ok])) <= tol


@pytest.mark.parametrize("most,segment", [(1, 1), (3, 2)])
@pytest.mark.parametrize("spot,value,state_type", [("x", float("inf"), None), ("x", float("nan"), "f16"), ("B", float("-inf"), None),
                                                   ("dt", float("nan"), None), ("state", float("inf"), "bf16")])
def test_emulated_values_that_are_not_finite_stay(emu_resident, emu_binary, tmp_path, monkeypatch, spot, value, state_type,  # noqa: F811
                                                  most, segment):
    wl, init = _sticky(spot, value, "cpu", 500, [1.0, 60.0, 20.0, 400.0])
    y_ref, st_ref, _ = _emulate(emu_binary, wl, init, tmp_path, 0, "end", state_type=state_type)
    monkeypatch.setenv("EMU_PIECES", str(most))
    monkeypatch.setenv("EMU_SEGMENTS", str(segment))
    for order, align in ((0, "end"), (1, "start")):
        y, st, _ = _emulate(emu_resident, wl, init, tmp_path, order, align, state_type=state_type)
        _same_finite(st.astype(np.float64), st_ref, 1e-2)
        _same_finite(y, y_ref, TOL["bf16"])


@pytest.mark.gpu
@pytest.mark.parametrize("spot", sorted(STICKY))
def test_gpu_values_that_are_not_finite_stay(spot):
    """9000 tokens, which this scan cuts, against three sequences of a third each that resume from the one before."""
    from helpers import gpu_run

    print(spot, flush=True)
    wl, init = _sticky(spot, float("inf"), "cuda:0", 9000, [1.0, 1.0, 30.0, 4.0])
    y, st, _ = gpu_run(wl, init)
    state, ys, states = init[0], [], []
    for lo in (0, 3000, 6000):
        part = [t[lo:lo + 3000].contiguous() for t in (wl.inputs.x, wl.inputs.dt, wl.inputs.B, wl.inputs.C)]
        at = [p - lo for p in wl.ckpt_pos[0] if lo < p <= lo + 3000]
        y1, st1, _ = gpu_run(wl, [state], inputs=type(wl.inputs)(*part), cu=np.asarray([0, 3000], np.int32),
                             ckpt_pos=[sorted({*at, 3000})])
        ys.append(y1)
        states += [st1[k] for k in range(len(at))]
        state = st1[-1].contiguous()
    _same_finite(st.cpu().numpy(), torch.stack(states).cpu().numpy(), 1e-2)
    _same_finite(y.float().cpu().numpy(), torch.cat(ys).float().cpu().numpy(), TOL["bf16"])


@pytest.mark.gpu
@pytest.mark.parametrize("what", SPOILED)
def test_gpu_values_that_are_not_finite(what):
    """300 equal sequences, a batch for this scan, against one alone, which the other scan takes."""
    from helpers import gpu_run

    print(what, flush=True)
    wl, init = _spoiled(what, "cuda:0", copies=300)
    one, first = _spoiled(what, "cuda:0")
    y_ref, st_ref, _ = gpu_run(one, first)
    y, st, _ = gpu_run(wl, init)
    y_ref, st_ref = y_ref.float().cpu().numpy(), st_ref.cpu().numpy()
    assert not np.isfinite(y_ref).all() and np.isfinite(st_ref).all() == (what[0] in "Cs" and "step_" not in what)
    y, st = y.float().cpu().numpy().reshape(300, *y_ref.shape), st.cpu().numpy().reshape(300, *st_ref.shape)
    for k in (0, 1, 137, 299):
        _same_reach(st[k], st_ref, 1e-3)
        _same_reach(y[k], y_ref, TOL["bf16"])


# A cached state that is updated in place: the initial state of a cut sequence is the slot of its only checkpoint.
def _in_place(shape, lens, device):
    total = sum(lens)
    wl = make_workload(2, device, seed=37, batch=1, len_range=(total, total), shape=shape)
    wl.seqlens, wl.cu_seqlens = list(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.ckpt_pos = [[n] for n in lens]
    g = torch.Generator(device=device).manual_seed(41)
    return wl, [torch.randn((shape.nheads, shape.headdim, 128), generator=g, device=device) for _ in lens]


@pytest.mark.parametrize("state_type", [None, "f16", "bf16"])
def test_emulated_states_updated_in_place(emu_resident, tmp_path, monkeypatch, state_type):
    """The workgroups run from the last to the first."""
    wl, init = _in_place(LayerShape(8, 64, 128, 2, 64, "bf16"), [200, 40, 131], "cpu")
    monkeypatch.setenv("EMU_PIECES", "1")
    monkeypatch.setenv("EMU_SEGMENTS", "1")
    want = _emulate(emu_resident, wl, init, tmp_path, 0, "end", state_type=state_type)[2]
    monkeypatch.setenv("EMU_LAST_BLOCK_FIRST", "1")
    monkeypatch.setenv("EMU_IN_PLACE", "1")
    assert np.array_equal(_emulate(emu_resident, wl, init, tmp_path, 0, "end", state_type=state_type)[2], want)


@pytest.mark.gpu
def test_gpu_states_updated_in_place():
    import paper_2411_19379_amd as ssm

    wl, init = _in_place(LayerShape(8, 64, 128, 2, 64, "bf16"), [5000, 90, 9000], "cuda:0")
    plan = ssm.Plan(8, 64, 128, 2, 64, "bf16", wl.cu_seqlens, wl.ckpt_pos)
    i = wl.inputs

    def run(states, out):
        y = torch.empty_like(i.x)
        ssm.prefill(plan, i.x, i.dt, wl.A, i.B, i.C, wl.D, states, y_out=y, state_out=out)
        torch.cuda.synchronize()
        return y

    apart = torch.empty((3, 8, 64, 128), device="cuda:0")
    want = run(init, apart)
    for rep in range(20):
        print(f"in place, pass {rep}", flush=True)
        states = torch.stack(init)
        assert torch.equal(run(list(states), states).view(torch.int16), want.view(torch.int16))
        assert torch.equal(states, apart)
    plan.close()


# on the GPU: batches that the plan gives to this scan, H, P, G, lengths, decay, type of the cached states; then pieces, segments,
# continued pieces and sums of segments
GPU_CASES = {
    # several rounds of uncut pieces
    "many_short": (32, 64, 2, [130, 65, 1, 64, 63, 0] * 48, 1.0, "f32", (240, 0, 0, 0)),
    # the same with tiles that leave the range of the masks' factors
    "many_short_strong_decay": (32, 64, 2, [130, 65, 1, 64, 63, 0] * 48, 60.0, "f32", (240, 0, 0, 0)),
    # pieces that start from segments
    "cut": (16, 64, 1, [33000], 1.0, "f32", (58, 57, 57, 7)),
    # whose segments all count
    "cut_slow_decay": (16, 64, 1, [17001, 9000], 0.01, "f32", (60, 58, 58, 7)),
    # and of which hardly any does
    "cut_strong_decay": (16, 64, 1, [33000], 60.0, "f32", (58, 57, 57, 7)),
    # 103 segments in front of the last piece, summed up in eights
    "sums_of_segments": (8, 64, 2, [33000], 0.01, "f32", (104, 103, 103, 12)),
    # pieces of more than 2000 tokens, in two segments, all of which count
    "long_pieces_slow_decay": (32, 64, 2, [67700], 0.002, "f32", (32, 62, 31, 7)),
    "p128_f16": (8, 128, 2, [20011, 15000], 1.0, "f16", (62, 60, 60, 7)),
    "p256_bf16": (4, 256, 1, [24000], 1.0, "bf16", (63, 62, 62, 7)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("case", sorted(GPU_CASES))
def test_gpu_matches_oracle(case):
    """Every head of every token and checkpoint.  The tolerances of reduced states add a rounding of the cached state and
    one of the checkpoint, as in the stretches' tests."""
    from helpers import gpu_run
    from test_gpu_configs import compare_all_heads

    H, P, G, lens, a_scale, state, walked = GPU_CASES[case]
    total = sum(lens)
    wl = make_workload(2, "cuda", seed=61, batch=1, len_range=(total, total), shape=LayerShape(H, P, 128, G, 64, "bf16"))
    wl.seqlens, wl.cu_seqlens = list(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wl.ckpt_pos = [sorted({max(1, n // 3), n}) if n else [] for n in lens]
    wl.A = wl.A * a_scale
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[state]
    init = [None if i % 2 else (0.5 * torch.randn(H, P, 128, device="cuda")).to(kind) for i in range(len(lens))]
    ref = [None if v is None else v.float().cpu().numpy() for v in init]
    import paper_2411_19379_amd as ssm
    plan = ssm.Plan(H, P, 128, G, 64, "bf16", wl.cu_seqlens, wl.ckpt_pos, state_dtype=state)
    assert plan.scan() == ("resident", *walked)
    plan.close()
    y, states, info = gpu_run(wl, init, state_dtype=state)
    compare_all_heads(wl, y, states.float(), ref, tol={"f32": TOL["bf16"], "f16": 2e-2, "bf16": 2.5e-2}[state], block=H)
