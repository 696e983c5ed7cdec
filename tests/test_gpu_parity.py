"""GPU parity tests: the HIP path through the C ABI against the fp64 oracle, element by element,
on the same seeded inputs.  Tolerances (per output tensor, max-norm relative): 1e-5 for f32 I/O,
2e-2 for bf16 I/O plus max-abs 5e-2 on h."""
import os

import numpy as np
import pytest
import torch

import parity_util as pu
from paper_2412_07752_amd import api, synth
from paper_2412_07752_amd.synth import CELL_ELMAN, CELL_GRU, CELL_GRU4, CELL_LSTM, CELL_SLSTM, Workload

pytestmark = pytest.mark.gpu
CELLS = [CELL_LSTM, CELL_GRU, CELL_SLSTM, CELL_ELMAN, CELL_GRU4]
PLAN_ENV = ("FLASHRNN_MULTI", "FLASHRNN_BT", "FLASHRNN_NWU", "FLASHRNN_KS", "FLASHRNN_GPAR", "FLASHRNN_SPIN_LIMIT", "FLASHRNN_DEEP_FETCH",
            "FLASHRNN_KIND", "FLASHRNN_RECOMPUTE_STEPS", "FLASHRNN_MESH", "FLASHRNN_SPLIT", "FLASHRNN_STEP")


@pytest.fixture(autouse=True)
def clean_env():
    for k in PLAN_ENV:
        os.environ.pop(k, None)
    os.environ["FLASHRNN_SPIN_LIMIT"] = "400000"
    yield
    for k in PLAN_ENV:
        os.environ.pop(k, None)


def _dlast(w, seed=99):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((w.S, w.B, w.NH, w.D)).astype(np.float32)


def _check(w, env=None, with_dlast=False, clip=None, elementwise=True):
    os.environ.update(env or {})
    print(f"case {w.name} env={env}", flush=True)
    inp = synth.make_inputs(w)
    dl = _dlast(w) if (with_dlast and w.backward) else None
    ref = pu.run_oracle(w, inp, dl, clip=clip)
    gpu = pu.run_gpu(w, inp, dl, clip=clip)
    res = pu.compare(w, gpu, ref)
    pu.assert_close(w, res)
    if elementwise:
        pu.assert_states_elementwise(w, gpu, ref)
    return gpu


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("dtype,D", [("bf16", 16), ("bf16", 32), ("bf16", 48), ("bf16", 64), ("bf16", 96), ("bf16", 128),
                                     ("bf16", 160), ("bf16", 192), ("f32", 16), ("f32", 48), ("f32", 64), ("f32", 96),
                                     ("f32", 128)])
def test_one_workgroup_per_group(cell, dtype, D):
    """Ragged batch (13 rows), several heads, non-zero initial states and final-state gradients."""
    w = Workload(f"single_{cell}_{dtype}_D{D}", cell, 9, 13, 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D)
    _check(w, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("bt", [16, 8, 4])
def test_batch_tiles(cell, bt):
    """Batch tiles of 16, 8 and 4 rows (idle MFMA lanes take over point-wise work); 21 rows = ragged last tile."""
    w = Workload(f"bt{bt}_{cell}", cell, 11, 21, 3, 64, "bf16", True, bias="forget3" if cell in (CELL_LSTM, CELL_SLSTM) else "uniform0.1",
                 init="uniform0.1", seed=bt)
    _check(w, {"FLASHRNN_BT": str(bt)}, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("dtype,D,env", [
    ("bf16", 64, {"FLASHRNN_NWU": "1"}), ("bf16", 64, {"FLASHRNN_NWU": "2"}), ("bf16", 128, {"FLASHRNN_NWU": "2"}),
    ("bf16", 192, {"FLASHRNN_NWU": "4"}), ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 256, {}), ("bf16", 384, {}),
    ("f32", 64, {"FLASHRNN_NWU": "1"}), ("f32", 128, {"FLASHRNN_KS": "4"}), ("f32", 192, {}), ("f32", 256, {}),
])
def test_groups_split_over_workgroups(cell, dtype, D, env):
    """A head served by several workgroups that exchange h (forward) / dg (backward) every step (full 16-row tiles)."""
    e = {"FLASHRNN_MULTI": "1", "FLASHRNN_BT": "16"}
    e.update(env)
    w = Workload(f"multi_{cell}_{dtype}_D{D}", cell, 10, 19, 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + 1)
    _check(w, e, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D,bt", [(64, 4), (64, 8), (112, 4), (128, 4), (128, 8), (160, 4), (192, 4)])
def test_staged_backward_kernels(cell, D, bt):
    """Every wave contracts all gate gradients of the head in one chain: heads that fill the contraction length and heads that pad it."""
    w = Workload(f"staged_{cell}_D{D}_bt{bt}", cell, 8, 10, 2, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + bt)
    _check(w, {"FLASHRNN_BT": str(bt)}, with_dlast=True)
    assert api.flashrnn_plan_kernel(api.make_desc(cell, 8, 10, 2, D, api.FLASHRNN_BF16), True) == (1, bt, 1)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("bt", [16, 8, 4])
@pytest.mark.parametrize("D", [48, 112])
def test_batch_tiles_with_f32_io(cell, bt, D):
    """f32 I/O (f32 MFMA, rel 1e-5): the same three tile heights; 21 rows = ragged last tile, head sizes that pad the contraction axis."""
    w = Workload(f"f32_bt{bt}_{cell}_D{D}", cell, 10, 21, 2, D, "f32", True, bias="forget3" if cell in (CELL_LSTM, CELL_SLSTM) else "uniform0.1",
                 init="uniform0.1", seed=bt + D)
    _check(w, {"FLASHRNN_BT": str(bt)}, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D", [16, 32, 80, 96, 128, 144, 192, 256])
def test_four_row_tiles_with_f32_io(cell, D):
    """4-row float32 tiles on the 4 x 4 matrix instruction: full and padded contraction quarters, one workgroup per group (up to 128
    units) and split groups (beyond); 7 rows = ragged last tile."""
    w = Workload(f"f32_quads_{cell}_D{D}", cell, 6, 7, 2, D, "f32", True, bias="uniform0.1", init="uniform0.1", seed=D + 5)
    _check(w, {"FLASHRNN_BT": "4"}, with_dlast=True)
    d = api.make_desc(cell, 6, 7, 2, D, api.FLASHRNN_F32)
    assert all(api.flashrnn_plan_kernel(d, x)[1] == 4 for x in (0, 1))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D,bt", [(32, 4), (32, 8), (64, 4), (64, 8), (16, 4), (48, 8), (48, 4)])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 13])
def test_backward_kernels_that_fetch_deep(cell, D, bt, T):
    """The backward kernels for inputs that come from HBM (taken by themselves only for sequences beyond the last-level cache):
    forced here on short sequences, every length around the depth of their pipeline."""
    w = Workload(f"deep_{cell}_D{D}_bt{bt}_T{T}", cell, T, 11, 2, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=T + D + bt)
    _check(w, {"FLASHRNN_DEEP_FETCH": "1", "FLASHRNN_BT": str(bt)}, with_dlast=True)
    assert api.flashrnn_plan_kernel(api.make_desc(cell, T, 11, 2, D, api.FLASHRNN_BF16), True)[0] == 2   # (that variant ran)


@pytest.mark.parametrize("D", [144, 160, 176])
def test_four_gate_gru_with_many_groups_takes_8_row_tiles_backward(D):
    """More groups of 4 rows than CUs: the staged 8-row backward kernel, which the planner takes only while it keeps every register
    (4 to 11 % faster than the 4-row one there)."""
    d = api.make_desc(CELL_GRU4, 3, 90, 12, D, api.FLASHRNN_BF16)
    assert api.flashrnn_plan_kernel(d, True) == (1, 8, 1)
    w = Workload(f"gru4_bt8_D{D}", CELL_GRU4, 3, 90, 12, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D)
    _check(w, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("bt", [8, 4])
def test_generic_kernels_on_small_batch_tiles(cell, bt):
    """The generic persistent kernels (lane-wise global accesses) on the shapes the staged tile kernels normally take."""
    w = Workload(f"generic_bt{bt}_{cell}", cell, 7, 11, 2, 96, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=bt + 40)
    _check(w, {"FLASHRNN_KIND": "0", "FLASHRNN_BT": str(bt)}, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
def test_forward_only_small_batch_tile(cell):
    """No gate cache: the staged forward kernel moves states only."""
    w = Workload(f"fwdonly_{cell}", cell, 6, 7, 2, 128, "bf16", False, bias="uniform0.1", init="uniform0.1", seed=77)
    _check(w)


@pytest.mark.parametrize("cell", [CELL_LSTM, CELL_GRU, CELL_SLSTM])
def test_forward_calls_with_and_without_saved_values_plan_apart(cell):
    """More groups than CUs (12 x 64 with 256 rows): the forward call that saves its values takes 4-row tiles, the one that
    saves nothing 8-row tiles (the sLSTM 4 rows either way); both against the oracle."""
    d = api.make_desc(cell, 3, 256, 12, 64, api.FLASHRNN_BF16)
    assert api.flashrnn_plan_kernel(d, 0)[:2] == (1, 4) and api.flashrnn_plan_kernel(d, 2)[:2] == (1, 4 if cell == CELL_SLSTM else 8)
    with pytest.raises(api.FlashRNNError):
        api.flashrnn_plan_kernel(d, 3)
    for backward in (False, True):
        _check(Workload(f"twoplans_{cell}_{int(backward)}", cell, 3, 256, 12, 64, "bf16", backward, bias="uniform0.1", init="uniform0.1", seed=91))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("clip", [0.0, 0.02, 1e6])
@pytest.mark.parametrize("dtype,D,env", [("bf16", 64, {}), ("bf16", 192, {}), ("bf16", 96, {"FLASHRNN_KIND": "0"}), ("f32", 32, {}),
                                         ("bf16", 128, {"FLASHRNN_MULTI": "1", "FLASHRNN_KS": "4"})])
def test_recurrent_gradient_clip(cell, clip, dtype, D, env):
    """Sec. 4.1: the R^T dg_t term clipped value by value after every step (0 cuts it; a huge bound changes nothing),
    in the tile, generic, f32 and split-group kernels.  (The recurrent term has values of a few tenths here: 0.02 bites.)"""
    w = Workload(f"clip{clip}_{cell}_{dtype}_D{D}", cell, 7, 6, 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + 3)
    os.environ.update(env)
    print(f"case {w.name} env={env}", flush=True)
    inp, dl = synth.make_inputs(w), _dlast(w)
    ref, ref_free = pu.run_oracle(w, inp, dl, clip=clip), pu.run_oracle(w, inp, dl)
    gpu = pu.run_gpu(w, inp, dl, clip=clip)
    # errors relative to the scale of the unclipped gradients (the clip shrinks values, not rounding errors) ...
    res = pu.compare(w, gpu, ref, scale_ref=ref_free)
    pu.assert_close(w, res)
    # ... and with an absolute bound: the unclipped run meets the tolerance as it is defined (relative to its own
    # reference), and clipping must not make any tensor's absolute error larger than twice that run's (or than the
    # plain tolerance on the clipped reference, whichever is larger)
    gpu_free = pu.run_gpu(w, inp, dl)
    res_free = pu.compare(w, gpu_free, ref_free)
    pu.assert_close(w, res_free)
    plain = pu.compare(w, gpu, ref)
    tol = pu.TOL_BF16_REL if dtype == "bf16" else pu.TOL_F32_REL
    for k, (r, a) in plain.items():
        assert r <= tol or a <= 2.0 * res_free[k][1] + 1e-30, f"{w.name} {k}: abs {a:.3e} vs unclipped run's {res_free[k][1]:.3e}"
    if clip == 0.02:   # the bound did change the result
        assert np.abs(ref_free["dWx"] - gpu["dWx"]).max() > 1e-3


@pytest.mark.parametrize("cell", [CELL_LSTM, CELL_GRU, CELL_SLSTM])
@pytest.mark.parametrize("dtype,D", [("bf16", 208), ("bf16", 320), ("bf16", 640), ("f32", 144), ("f32", 208)])
def test_split_groups_with_padded_contraction(cell, dtype, D):
    """Head sizes between the instantiated contraction lengths: the exchanged rows and the packed R are zero beyond D."""
    w = Workload(f"pad_{cell}_{dtype}_D{D}", cell, 5, 5, 1 if D > 400 else 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D)
    _check(w, with_dlast=True)


def test_largest_head_takes_a_whole_xcd():
    """D = 1024 in one head: a group is 32 workgroups (every CU of one XCD) x 2 unit waves x 4 contraction slices; the five
    batch rows make two groups of batch tile 4, on two XCDs."""
    w = Workload("lstm_D1024", CELL_LSTM, 4, 5, 1, 1024, "bf16", True, seed=9)
    _check(w)
    d = api.make_desc(CELL_LSTM, 4, 5, 1, 1024, api.FLASHRNN_BF16)
    assert api.flashrnn_plan(d)[0] == 64 and api.flashrnn_plan_kernel(d)[2] == 32


def test_backward_groups_take_whole_xcds_and_the_whole_chip_where_they_need_them():
    """A head of 1024 units needs every CU of an XCD per group in both directions (four 4-row groups of a 16-row batch side by
    side, not one 16-row group); two 8-row groups of a 2048-unit head need all 256 CUs."""
    d = api.make_desc(CELL_LSTM, 8, 16, 1, 1024, api.FLASHRNN_BF16)
    for bwd in (False, True):
        staged, bt, split = api.flashrnn_plan_kernel(d, bwd)
        assert (staged, bt, split) == (0, 4, 32) and api.flashrnn_plan(d, bwd)[0] == 128
    d = api.make_desc(CELL_LSTM, 8, 16, 1, 2048, api.FLASHRNN_BF16)
    assert api.flashrnn_plan_kernel(d, True)[1:] == (8, 128) and api.flashrnn_plan(d, True)[0] == 256
    w = Workload("lstm_D1024_B16", CELL_LSTM, 5, 16, 1, 1024, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=10)
    _check(w, with_dlast=True)


@pytest.mark.parametrize("cell,D,B,NH", [(CELL_LSTM, 1040, 5, 1), (CELL_LSTM, 1280, 19, 1), (CELL_LSTM, 1536, 6, 2), (CELL_LSTM, 2048, 9, 1),
                                         (CELL_LSTM, 2688, 5, 1), (CELL_SLSTM, 1536, 7, 1), (CELL_SLSTM, 2048, 16, 1), (CELL_GRU, 1280, 12, 1),
                                         (CELL_GRU, 2688, 3, 1), (CELL_ELMAN, 2048, 4, 1), (CELL_GRU4, 1536, 4, 1)])
def test_heads_beyond_one_xcd_are_spread_over_the_chip(cell, D, B, NH):
    """Heads of more than 1024 units (App. H.1 quotes 2688 as the largest fused head on the paper's GPU): R does not fit the
    registers of one XCD's CUs, so a group's workgroups sit on all eight XCDs and exchange h / dg through memory."""
    w = Workload(f"spread_{cell}_D{D}", cell, 5, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + B)
    _check(w, with_dlast=True)
    d = api.make_desc(cell, 5, B, NH, D, api.FLASHRNN_BF16)
    for bwd in (False, True):
        assert api.flashrnn_plan_kernel(d, bwd)[2] == D // 16


@pytest.mark.parametrize("cell", CELLS)
def test_spread_groups_loop_when_they_do_not_fit(cell):
    """The spread placement forced onto a small head, two groups in flight out of nine: workgroups loop over groups."""
    w = Workload(f"spreadloop_{cell}", cell, 6, 33, 1, 64, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=6)
    _check(w, {"FLASHRNN_MULTI": "2", "FLASHRNN_GPAR": "2"}, with_dlast=True)


@pytest.mark.parametrize("cell,NH,D", [(CELL_LSTM, 32, 128), (CELL_GRU, 24, 144), (CELL_SLSTM, 12, 144)])
def test_weight_gradient_gemm_with_large_tiles(cell, NH, D):
    """Many heads: the dR GEMM takes its 128 x 256 tile (ragged in both directions at D = 144; GRU: the candidate column of B comes
    from the recurrent-side gradient buffer), and the contraction over (t, b) has a ragged last round."""
    w = Workload(f"widegemm_{cell}_NH{NH}_D{D}", cell, 7, 5, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=NH + D)
    _check(w, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
def test_group_loop_when_groups_do_not_fit(cell):
    """More groups than run at once: workgroups loop over groups and reload R per head."""
    w = Workload(f"loop_{cell}", cell, 7, 40, 3, 64, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=5)
    _check(w, {"FLASHRNN_MULTI": "1", "FLASHRNN_NWU": "2", "FLASHRNN_GPAR": "4"}, with_dlast=True)


@pytest.mark.parametrize("cell,NH,D,B,bt,split", [
    (CELL_SLSTM, 8, 256, 66, 4, 2), (CELL_SLSTM, 3, 224, 177, 4, 2), (CELL_LSTM, 8, 256, 130, 8, 2), (CELL_SLSTM, 1, 768, 65, 8, 24), (CELL_SLSTM, 2, 1024, 33, 8, 32),
])
def test_backward_groups_in_rounds_of_smaller_tiles(cell, NH, D, B, bt, split):
    """Batches whose 16-row tiles would run at once, or in fewer rounds, in kernels that are slower all the same; ragged last tiles."""
    w = Workload(f"rounds_{cell}_D{D}", cell, 5, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=B)
    _check(w, with_dlast=True)
    d = api.make_desc(cell, 5, B, NH, D, api.FLASHRNN_BF16)
    assert api.flashrnn_plan_kernel(d, True)[1:] == (bt, split)


def _with_roles(cell, T, B, NH, D, backward):
    """(waves, workgroups per group) of a plan that must have wave roles: 12 waves where the partial sums meet in LDS or three k-steps share eight waves
    of a mesh, 8 waves and 64 units per workgroup where each wave waits for its own lanes, 8 and 32 in the mesh of an XCD."""
    os.environ["FLASHRNN_SPLIT"] = "3" if backward is True else "2"
    d = api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16)
    return api.flashrnn_plan(d, backward)[2], api.flashrnn_plan_kernel(d, backward)[2]


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,bt,B,T", [
    (2, 256, 4, 7, 13), (1, 256, 8, 9, 1), (1, 320, 4, 5, 3), (3, 320, 8, 8, 2), (1, 384, 4, 6, 7),   # each compute wave waits for its own lanes' words
    (2, 208, 4, 5, 8), (1, 272, 8, 11, 7), (1, 448, 4, 6, 13), (1, 640, 8, 9, 5), (1, 768, 4, 5, 2), (1, 208, 16, 17, 6),   # sums via LDS; 13, 17, 28 output blocks over 8 waves
    (2, 64, 8, 40, 3),   # a small head, groups in rounds
])
def test_backward_of_split_heads_exchanges_partial_sums(cell, NH, D, bt, B, T):
    """Kernels with wave roles: sequences shorter and longer than the ring of inputs, ragged batches, output blocks that do not fill the waves."""
    w = Workload(f"partial_{cell}_D{D}", cell, T, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + bt)
    env = {"FLASHRNN_MULTI": "1", "FLASHRNN_BT": str(bt)}
    if D == 64:
        env["FLASHRNN_GPAR"] = "8"
    _check(w, env, with_dlast=True)
    direct = D == 320 or (D in (256, 384) and bt == 4)
    if cell != CELL_ELMAN or direct:   # (Elman: one gate's gradients are less to exchange than partial sums)
        assert _with_roles(cell, T, B, NH, D, True) == ((8, D // 64) if direct else (12, D // 32 if D % 32 == 0 else D // 16))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,B,T,env", [
    (2, 256, 9, 19, {"FLASHRNN_MULTI": "1", "FLASHRNN_MESH": "1", "FLASHRNN_BT": "8"}), (1, 384, 5, 3, {"FLASHRNN_MULTI": "1", "FLASHRNN_MESH": "1", "FLASHRNN_BT": "4"}),
    (1, 768, 20, 5, {"FLASHRNN_MESH": "1", "FLASHRNN_BT": "16"}), (1, 896, 11, 37, {"FLASHRNN_BT": "8"}), (1, 1024, 17, 4, {"FLASHRNN_BT": "16"}),
    (1, 1536, 16, 35, {}), (3, 128, 13, 7, {"FLASHRNN_MULTI": "2", "FLASHRNN_BT": "8", "FLASHRNN_GPAR": "3"}), (1, 256, 3, 41, {"FLASHRNN_MULTI": "2", "FLASHRNN_BT": "4"}), (1, 2048, 7, 1, {}),
])
def test_backward_of_split_heads_in_two_hand_overs(cell, NH, D, B, T, env):
    """Subgroups of 1 to 16 members, inside one XCD (two blocks of 16 units per member) and one subgroup per XCD; contractions that do not fill the
    waves' k-steps, ragged batches, groups in rounds, sequences shorter and longer than the ring of inputs."""
    w = Workload(f"mesh_{cell}_D{D}", cell, T, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + B)
    _check(w, env, with_dlast=True)
    spread = D > 1024 or env.get("FLASHRNN_MULTI") == "2"
    if cell != CELL_ELMAN or spread:   # (inside an XCD Elman exchanges gate gradients)
        assert _with_roles(cell, T, B, NH, D, True) == ((8, D // 32) if not spread else (12 if w.G * D // 8 <= 768 else 8, D // 16))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,bt,B,T,split", [
    (1, 256, 4, 5, 75, 16), (8, 256, 4, 32, 37, 4), (1, 512, 8, 7, 41, 32), (1, 736, 16, 17, 34, 23), (1, 1024, 4, 3, 35, 32), (2, 384, 16, 30, 50, 24),
])
def test_split_heads_over_many_steps(cell, NH, D, bt, B, T, split):
    """Sequences longer than the rings of inputs in LDS (the slots are used again), few and many members per group, contraction slices that the head
    does not fill, half steps."""
    w = Workload(f"ring_{cell}_D{D}", cell, T, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + T)
    _check(w, {"FLASHRNN_BT": str(bt)}, with_dlast=True)
    assert api.flashrnn_plan_kernel(api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16))[2] == split


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,B", [(2, 16, 1), (3, 48, 1), (1, 112, 5), (2, 192, 13), (1, 272, 1), (1, 768, 33), (1, 1024, 2)])
def test_one_step_calls(cell, NH, D, B):
    """T = 1 on the kernel of its own: contractions that are no multiple of the threads' rounds, ragged batch tiles, with and without saved values
    and initial states, and the backward call behind it."""
    d = api.make_desc(cell, 1, B, NH, D, api.FLASHRNN_BF16)
    assert api.flashrnn_plan(d) == ((B + 3) // 4 * NH * (D // 16) if B > 1 else NH * (D // 16), (B + 3) // 4 * (D // 16) if B > 1 else D // 16, 4)
    for init in ("uniform0.1", "zero"):
        _check(Workload(f"step_{cell}_D{D}_{init}", cell, 1, B, NH, D, "bf16", True, bias="uniform0.1", init=init, seed=D + B), with_dlast=True)
    _check(Workload(f"step_{cell}_D{D}_infer", cell, 1, B, NH, D, "bf16", False, bias="uniform0.1", init="uniform0.1", seed=D))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,B", [(4, 192, 1), (2, 96, 5), (1, 768, 3), (1, 1152, 2)])
def test_one_step_calls_that_carry_their_states_in_place(cell, NH, D, B):
    """states0 = states[1] of the same buffer, call after call: every unit's new state must come from the old h of the whole head."""
    w = Workload(f"carry_{cell}_D{D}", cell, 6, B, NH, D, "bf16", False, bias="uniform0.1", init="uniform0.1", seed=D + B)
    inp = synth.make_inputs(w)
    print(f"case {w.name}", flush=True)
    ref = pu.run_oracle(w, inp)
    Wx, R, b = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b"))
    d = api.make_desc(cell, 1, B, NH, D, api.FLASHRNN_BF16)
    ws = api.alloc_workspace(d, "cuda")
    states = torch.empty((2, w.S, B, NH, D), dtype=torch.float32, device="cuda")
    for scratch in (False, True):
        states[1].copy_(pu.to_device(inp["states0"], "f32"))
        steps = [states[1].clone()]
        for t in range(w.T):
            if scratch:
                api.flashrnn_fwd_static_scratch(cell, Wx[t:t + 1], R, b, states[1], save_for_backward=False, states=states)
                api.flashrnn_check(d, api.STATIC_SCRATCH)
            else:
                api.flashrnn_fwd(cell, Wx[t:t + 1], R, b, states[1], save_for_backward=t % 2 == 1, workspace=ws, states=states)
                api.flashrnn_check(d, ws)
            assert torch.equal(states[0], steps[-1])   # slot 0 holds what the call started from
            steps.append(states[1].clone())
        gpu = {"states": pu.to_host64(torch.stack(steps))}
        pu.assert_close(w, pu.compare(w, gpu, ref))
        pu.assert_states_elementwise(w, gpu, ref)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("dtype,NH,D,B", [("bf16", 2, 64, 7), ("bf16", 1, 192, 19), ("bf16", 2, 256, 9), ("bf16", 1, 768, 35), ("bf16", 1, 1152, 5), ("f32", 2, 96, 7), ("f32", 1, 208, 5)])
def test_initial_states_in_a_slot_of_the_output(cell, dtype, NH, D, B):
    """states0 = any slot of `states`: the same bits as with a buffer of its own, in every kernel family."""
    w = Workload(f"slot_{cell}_{dtype}_D{D}", cell, 3, B, NH, D, dtype, False, bias="uniform0.1", init="uniform0.1", seed=D + B)
    inp = synth.make_inputs(w)
    print(f"case {w.name}", flush=True)
    Wx, R, b = (pu.to_device(inp[k], dtype) for k in ("Wx", "R", "b"))
    s0 = pu.to_device(inp["states0"], "f32")
    ref, _, ws = api.flashrnn_fwd(cell, Wx, R, b, s0, save_for_backward=False)
    for slot in range(w.T + 1):
        states = torch.empty_like(ref)
        states[slot].copy_(s0)
        api.flashrnn_fwd(cell, Wx, R, b, states[slot], save_for_backward=False, workspace=ws, states=states)
        api.flashrnn_check(api.make_desc(cell, w.T, B, NH, D, api.FLASHRNN_BF16 if dtype == "bf16" else api.FLASHRNN_F32), ws)
        assert torch.equal(states, ref), slot


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,B", [(2, 96, 1), (1, 768, 3)])
def test_one_step_calls_from_zero_states_with_weights_that_are_not_finite(cell, NH, D, B):
    """No initial states: h_0 is zero, and zero times an infinite or NaN weight is NaN, as on the kernels of longer sequences."""
    w = Workload(f"zero_{cell}_D{D}", cell, 1, B, NH, D, "bf16", False, bias="uniform0.1", init="zero", seed=D + B)
    inp = synth.make_inputs(w)
    inp["R"][0, 3, 0, 5], inp["R"][NH - 1, D - 1, w.G - 1, D - 1] = np.inf, np.nan
    Wx, R, b = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b"))
    two = torch.cat([Wx, Wx])
    got, ref = (pu.to_host64(api.flashrnn_fwd(cell, x, R, b, save_for_backward=False)[0][1]) for x in (Wx, two))
    assert np.isnan(ref[0, :, 0, 5]).all() and np.isnan(ref).sum() <= 2 * w.S * B
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    fin = np.isfinite(ref)
    assert np.abs(got[fin] - ref[fin]).max() <= pu.TOL_BF16_REL * np.abs(ref[fin]).max()


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("T", [0, 1, 2, 3])
def test_degenerate_lengths(cell, T):
    """The staged kernels look two steps ahead: the shortest sequences take every clamped branch of that."""
    w = Workload(f"T{T}_{cell}", cell, T, 5, 2, 32, "bf16", True, bias="uniform0.1", init="uniform0.1")
    gpu = _check(w, with_dlast=True)
    if T == 0:
        assert np.all(gpu["dR"] == 0) and np.all(gpu["db"] == 0)


def test_large_single_head_split_with_contraction_slices():
    """D = 768 in one head (R is 4.7 MB): 24 workgroups x 2 unit waves x 4 contraction slices per group; with batch tiles
    of 4 rows the 16 rows make 4 groups, one per XCD."""
    w = Workload("lstm_D768", CELL_LSTM, 12, 16, 1, 768, "bf16", True, seed=3)
    _check(w)
    d = api.make_desc(CELL_LSTM, 12, 16, 1, 768, api.FLASHRNN_BF16)
    wg, per_head, waves = api.flashrnn_plan(d)
    staged, bt, split = api.flashrnn_plan_kernel(d)
    assert (wg, per_head, waves) == (96, 96, 8) and (staged, bt, split) == (False, 4, 24)
    _check(w, {"FLASHRNN_BT": "16"})
    assert api.flashrnn_plan(d) == (24, 24, 8)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("bt", [8, 4])
@pytest.mark.parametrize("dtype,D,env", [("bf16", 256, {}), ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 64, {"FLASHRNN_NWU": "1"})])
def test_split_groups_on_small_batch_tiles(cell, bt, dtype, D, env):
    """A head split over workgroups with batch tiles of 8 and 4 rows: fewer rows to exchange per group, lanes collect the four
    units of an exchange word from their neighbours before publishing."""
    e = {"FLASHRNN_MULTI": "1", "FLASHRNN_BT": str(bt)}
    e.update(env)
    w = Workload(f"multibt{bt}_{cell}_D{D}", cell, 9, 13, 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + bt)
    _check(w, e, with_dlast=True)


@pytest.mark.parametrize("dtype,D,env", [
    ("bf16", 256, {}), ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 64, {"FLASHRNN_MULTI": "2", "FLASHRNN_BT": "8"}), ("f32", 192, {}),
])
def test_split_groups_pass_every_nan_pattern_on(dtype, D, env):
    """The exchange buffers of a split head mark a missing word by the NaN of all ones: that value in a caller's data must reach the
    other workgroups as a NaN (no wait that never ends), and leave the other batch rows as they are, bit for bit."""
    e = {"FLASHRNN_MULTI": "1", "FLASHRNN_BT": "4"}
    e.update(env)
    os.environ.update(e)
    w = Workload(f"nan_{dtype}_D{D}", CELL_LSTM, 9, 8, 1, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D)
    inp = synth.make_inputs(w)
    ones = np.array([0xFFFFFFFF], dtype=np.uint32).view(np.float32)[0]
    bad = {k: None if v is None else v.copy() for k, v in inp.items()}
    bad["states0"][0, 2] = ones          # h_0 of row 2
    bad["dH"][5, 5, 0] = ones            # a gradient of row 5
    got, ref = pu.run_gpu(w, bad), pu.run_gpu(w, inp)   # (flashrnn_check after every call: no time-out)
    assert np.isnan(got["states"][1:, :, 2]).all()
    # The gates behind the cell state (i, f, z) carry the NaN from step to step; the output gate sees it through the recurrent term, whose
    # bound (infinite here) makes an infinity of a NaN.
    assert np.isnan(got["dWx"][:6, 5, :3]).all() and np.isnan(got["dWx"][5, 5]).all() and not np.isfinite(got["dWx"][:5, 5, 3]).any()
    rows = [r for r in range(8) if r != 2]
    assert np.array_equal(got["states"][:, :, rows], ref["states"][:, :, rows])
    rows.remove(5)
    assert np.array_equal(got["dWx"][:, rows], ref["dWx"][:, rows]) and np.array_equal(got["dstates0"][:, rows], ref["dstates0"][:, rows])


LARGE_CASES = [
    # (dtype, D, environment, batch): staged tile kernels, generic kernels, a head split over workgroups (with and
    # without contraction slices), f32 single and split
    ("bf16", 64, {}, 13), ("bf16", 192, {}, 6), ("bf16", 96, {"FLASHRNN_KIND": "0", "FLASHRNN_BT": "4"}, 9),
    ("bf16", 64, {"FLASHRNN_BT": "16"}, 19), ("bf16", 256, {}, 7), ("bf16", 128, {"FLASHRNN_MULTI": "1", "FLASHRNN_KS": "4"}, 18),
    ("f32", 64, {}, 5), ("f32", 192, {}, 6),
]


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("init", ["uniform0.1_bounded", "zero"])
@pytest.mark.parametrize("dtype,D,env,B", LARGE_CASES)
def test_saturated_gates(cell, init, dtype, D, env, B):
    """Finite pre-activations far out in both tails (a third of all Wx entries shifted by +-50, +-100, +-200, on every
    gate), non-zero R, 12 steps so that the sLSTM stabilizer is carried through jumps in both directions: the regime m
    exists for (App. A).  Nothing may overflow, underflow into a wrong branch or turn into NaN, forward or backward.
    Non-zero initial states respect the cell's invariant |c| <= n (|h| <= 1): bf16 rounding of an h of 100 and more would
    move pre-activations by tenths.  With f32 I/O the element-wise check of the sLSTM states is left to the max-norm one:
    the stabilizer reaches 230 here, where one float32 ulp is 1.5e-5, and every weight exp(. - m) carries that as a
    relative error, so single elements sit at 1e-5 to 2e-5."""
    w = Workload(f"sat_{cell}_{dtype}_D{D}_{init}", cell, 12, B, 2, D, dtype, True, bias="forget3" if cell in (CELL_LSTM, CELL_SLSTM) else "uniform0.1",
                 init=init, seed=D + B, wx="large_mix")
    gpu = _check(w, env, with_dlast=True, elementwise=not (cell == CELL_SLSTM and dtype == "f32"))
    for k, v in gpu.items():
        assert np.all(np.isfinite(v)), k


def test_forward_timeout_survives_the_backward_call():
    """A split plan whose forward waits gave up: the backward call that follows runs with a normal limit, and one check
    after it still reports the forward timeout (the two passes keep separate error words; only a forward call clears both)."""
    w = Workload("sticky", CELL_LSTM, 6, 16, 1, 64, "bf16", True)
    inp = synth.make_inputs(w)
    os.environ.update({"FLASHRNN_MULTI": "1", "FLASHRNN_NWU": "1", "FLASHRNN_SPIN_LIMIT": "-1"})
    Wx, R, b, dH = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b", "dH"))
    desc = api.make_desc(w.cell, w.T, w.B, w.NH, w.D, api.FLASHRNN_BF16)
    states, cache, ws = api.flashrnn_fwd(w.cell, Wx, R, b)
    os.environ["FLASHRNN_SPIN_LIMIT"] = "400000"
    api.flashrnn_bwd(w.cell, R, b, states, cache, dH, workspace=ws)
    with pytest.raises(api.FlashRNNError) as ei:
        api.flashrnn_check(desc, ws)
    assert ei.value.status == api.FLASHRNN_ERR_TIMEOUT
    # the next forward / backward pair on the same workspace is clean and correct again
    ref = pu.run_oracle(w, inp)
    states, cache, ws = api.flashrnn_fwd(w.cell, Wx, R, b, workspace=ws)
    dWx, dR, db, ds0 = api.flashrnn_bwd(w.cell, R, b, states, cache, dH, workspace=ws)
    api.flashrnn_check(desc, ws)
    gpu = {"states": pu.to_host64(states), "dWx": pu.to_host64(dWx), "dR": pu.to_host64(dR), "db": pu.to_host64(db), "dstates0": pu.to_host64(ds0)}
    pu.assert_close(w, pu.compare(w, gpu, ref))


def test_seeded_random_shapes():
    """A seeded sweep over (cell, dtype, T, B, NH, D, forward-only / backward, clip, initial states, final-state gradients)
    with whatever plan the library picks for each shape; stops at the first mismatch and names the case."""
    import random
    rng = random.Random(20241207)
    for it in range(48):
        cell = rng.choice(CELLS)
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        D = 16 * rng.choice([1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 16, 20, 24] if dtype == "bf16" else [1, 2, 3, 4, 6, 8, 12, 16])
        NH = rng.choice([1, 2, 3, 5, 8, 20])
        B = rng.choice([1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 33, 64])
        T = rng.choice([1, 2, 3, 4, 5, 8, 13])
        while NH * B * D * T > 400000 and B > 1:
            B = max(1, B // 2)
        bw = rng.random() < 0.8
        clip = rng.choice([None, None, 0.05, 0.0]) if bw else None
        w = Workload(f"rand{it}", cell, T, B, NH, D, dtype, bw, bias="uniform0.1", init=rng.choice(["zero", "uniform0.1"]), seed=it + 1000)
        print(f"case {it}: cell {cell} {dtype} T {T} B {B} NH {NH} D {D} bwd {bw} clip {clip}", flush=True)
        inp = synth.make_inputs(w)
        dl = _dlast(w, seed=it) if (bw and rng.random() < 0.5) else None
        ref = pu.run_oracle(w, inp, dl, clip=clip)
        free = pu.run_oracle(w, inp, dl) if clip is not None else None
        gpu = pu.run_gpu(w, inp, dl, clip=clip)
        pu.assert_close(w, pu.compare(w, gpu, ref, scale_ref=free))
        pu.assert_states_elementwise(w, gpu, ref)


RECOMPUTE_CASES = [
    # (dtype, D, B, T, environment): staged tile kernels, generic kernels, a head split over workgroups, f32; windows of 4 steps
    # (T = 11: a ragged first window), of one step, and the whole sequence in one window
    ("bf16", 64, 13, 11, {"FLASHRNN_RECOMPUTE_STEPS": "4"}), ("bf16", 192, 6, 9, {"FLASHRNN_RECOMPUTE_STEPS": "1"}),
    ("bf16", 96, 19, 11, {"FLASHRNN_RECOMPUTE_STEPS": "4", "FLASHRNN_KIND": "0", "FLASHRNN_BT": "16"}), ("bf16", 256, 7, 11, {"FLASHRNN_RECOMPUTE_STEPS": "3"}),
    ("bf16", 80, 5, 7, {}), ("f32", 48, 9, 10, {"FLASHRNN_RECOMPUTE_STEPS": "4"}), ("f32", 192, 5, 6, {"FLASHRNN_RECOMPUTE_STEPS": "2"}),
    # ... and the backward kernels that fetch deep, in windows of 5 steps (a ragged first window of 3)
    ("bf16", 64, 13, 13, {"FLASHRNN_RECOMPUTE_STEPS": "5", "FLASHRNN_DEEP_FETCH": "1"}),
]


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("dtype,D,B,T,env", RECOMPUTE_CASES)
def test_backward_with_recomputed_values(cell, dtype, D, B, T, env):
    """flashrnn_bwd_recompute: forward without a gate cache, backward from Wx and the states alone, window by window
    (carried state gradients, db sums and the GRU's recurrent-side gradients cross the window boundaries)."""
    os.environ.update(env)
    w = Workload(f"recompute_{cell}_{dtype}_D{D}", cell, T, B, 2, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + T)
    print(f"case {w.name} env={env}", flush=True)
    inp, dl = synth.make_inputs(w), _dlast(w)
    ref = pu.run_oracle(w, inp, dl)
    Wx, R, b, dH = (pu.to_device(inp[k], dtype) for k in ("Wx", "R", "b", "dH"))
    s0, dlast = pu.to_device(inp["states0"], "f32"), pu.to_device(dl, "f32")
    states, cache, ws = api.flashrnn_fwd(cell, Wx, R, b, s0, save_for_backward=False)
    assert cache is None
    dWx, dR, db, ds0, ws2 = api.flashrnn_bwd_recompute(cell, Wx, R, b, states, dH, dlast)
    desc = api.make_desc(cell, T, B, 2, D, api.FLASHRNN_BF16 if dtype == "bf16" else api.FLASHRNN_F32)
    api.flashrnn_check(desc, ws2)
    gpu = {"states": pu.to_host64(states), "dWx": pu.to_host64(dWx), "dR": pu.to_host64(dR), "db": pu.to_host64(db), "dstates0": pu.to_host64(ds0)}
    pu.assert_close(w, pu.compare(w, gpu, ref))


def test_backward_with_recomputed_values_empty_sequence():
    w = Workload("recompute_T0", CELL_SLSTM, 0, 5, 2, 32, "bf16", True, bias="uniform0.1", init="uniform0.1")
    inp, dl = synth.make_inputs(w), _dlast(w)
    ref = pu.run_oracle(w, inp, dl)
    Wx, R, b, dH = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b", "dH"))
    states, _, _ = api.flashrnn_fwd(w.cell, Wx, R, b, pu.to_device(inp["states0"], "f32"), save_for_backward=False)
    dWx, dR, db, ds0, _ = api.flashrnn_bwd_recompute(w.cell, Wx, R, b, states, dH, pu.to_device(dl, "f32"))
    gpu = {"states": pu.to_host64(states), "dWx": pu.to_host64(dWx), "dR": pu.to_host64(dR), "db": pu.to_host64(db), "dstates0": pu.to_host64(ds0)}
    pu.assert_close(w, pu.compare(w, gpu, ref))


def test_runs_are_bitwise_reproducible():
    """No float atomics anywhere: two runs give identical bits (single and split groups)."""
    for env in ({}, {"FLASHRNN_MULTI": "1", "FLASHRNN_NWU": "1"}):
        os.environ.update(env)
        w = Workload("repro", CELL_SLSTM, 16, 16, 2, 64, "bf16", True, bias="forget3", init="uniform0.1")
        inp = synth.make_inputs(w)
        a = pu.run_gpu(w, inp)
        b = pu.run_gpu(w, inp)
        for k in a:
            assert np.array_equal(a[k], b[k]), k


def test_chunked_sequence_equals_one_call():
    """states0 in / last states out: T1 steps then T2 steps from the saved states == T1 + T2 steps (f32 path, exact)."""
    w = Workload("chunk", CELL_SLSTM, 12, 8, 2, 32, "f32", False, bias="forget3", init="uniform0.1")
    inp = synth.make_inputs(w)
    Wx, R, b = (pu.to_device(inp[k], "f32") for k in ("Wx", "R", "b"))
    s0 = pu.to_device(inp["states0"], "f32")
    full, _, _ = api.flashrnn_fwd(w.cell, Wx, R, b, s0, save_for_backward=False)
    a, _, _ = api.flashrnn_fwd(w.cell, Wx[:7].contiguous(), R, b, s0, save_for_backward=False)
    c, _, _ = api.flashrnn_fwd(w.cell, Wx[7:].contiguous(), R, b, a[7].contiguous(), save_for_backward=False)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat([a, c[1:]]), full)


def test_exchange_timeout_is_reported_not_hung():
    """Negative spin limit: every cross-CU wait gives up at once, every kernel still runs to its end,
    flashrnn_check reports the timeout, and the next call with a normal limit is correct again."""
    w = Workload("timeout", CELL_LSTM, 6, 16, 1, 64, "bf16", False)
    inp = synth.make_inputs(w)
    os.environ.update({"FLASHRNN_MULTI": "1", "FLASHRNN_NWU": "1", "FLASHRNN_SPIN_LIMIT": "-1"})
    with pytest.raises(api.FlashRNNError) as ei:
        pu.run_gpu(w, inp)
    assert ei.value.status == api.FLASHRNN_ERR_TIMEOUT
    os.environ["FLASHRNN_SPIN_LIMIT"] = "400000"
    ref = pu.run_oracle(w, inp)
    pu.assert_close(w, pu.compare(w, pu.run_gpu(w, inp), ref))


def test_binding_rejects_wrong_shapes_and_dtypes():
    dev = "cuda"
    Wx = torch.zeros((4, 2, 4, 1, 32), dtype=torch.bfloat16, device=dev)
    R = torch.zeros((1, 32, 4, 32), dtype=torch.bfloat16, device=dev)
    b = torch.zeros((1, 4, 32), dtype=torch.bfloat16, device=dev)
    with pytest.raises(ValueError):
        api.flashrnn_fwd(CELL_LSTM, Wx, R[:, :16].contiguous(), b)
    with pytest.raises(ValueError):
        api.flashrnn_fwd(CELL_LSTM, Wx, R.float(), b)
    with pytest.raises(ValueError):
        api.flashrnn_fwd(CELL_GRU, Wx, R, b)
    with pytest.raises(TypeError):
        api.flashrnn_fwd(CELL_LSTM, Wx.half(), R.half(), b.half())
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=dev)
    d = api.make_desc(CELL_LSTM, 4, 2, 1, 32, api.FLASHRNN_BF16)
    import ctypes
    st = torch.empty((5, 2, 2, 1, 32), dtype=torch.float32, device=dev)
    rc = api.lib().flashrnn_fwd(ctypes.byref(d), Wx.data_ptr(), R.data_ptr(), b.data_ptr(), None, st.data_ptr(), None,
                                ws.data_ptr() + 8, None)
    assert rc == api.FLASHRNN_ERR_WORKSPACE


@pytest.mark.parametrize("D", [64, 256])
def test_forward_backward_replay_from_a_hip_graph(D):
    """The two entry points allocate nothing and record only kernels, so a caller may capture them.  The graph is replayed
    several times, with eager work and synchronizations in between, on changing inputs; every replay must reproduce the eager
    result bit for bit (one workgroup per group, and a head split over workgroups with its exchange buffers)."""
    w = Workload(f"graph_D{D}", CELL_SLSTM, 12, 8, 2, D, "bf16", True, bias="forget3", init="uniform0.1", seed=D)
    inp = synth.make_inputs(w)
    Wx, R, b = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b"))
    s0, dH = pu.to_device(inp["states0"], "f32"), pu.to_device(inp["dH"], "bf16")
    desc = api.make_desc(w.cell, w.T, w.B, w.NH, w.D, api.FLASHRNN_BF16)
    ws = api.alloc_workspace(desc, "cuda")
    states = torch.empty((w.T + 1, w.S, w.B, w.NH, w.D), dtype=torch.float32, device="cuda")
    cache = torch.empty(api.flashrnn_gate_cache_bytes(desc), dtype=torch.uint8, device="cuda")
    out = (torch.empty((w.T, w.B, w.G, w.NH, w.D), dtype=torch.bfloat16, device="cuda"), torch.empty((w.NH, w.D, w.G, w.D), device="cuda"),
           torch.empty((w.NH, w.G, w.D), device="cuda"), torch.empty((w.S, w.B, w.NH, w.D), device="cuda"))

    def step():
        api.flashrnn_fwd(w.cell, Wx, R, b, s0, workspace=ws, states=states, gate_cache=cache)
        api.flashrnn_bwd(w.cell, R, b, states, cache, dH, None, workspace=ws, out=out)

    def snapshot():
        torch.cuda.synchronize()
        return [t.clone() for t in (states,) + out]

    step()                       # warm-up outside the capture (kernel attributes are set on first use)
    api.flashrnn_check(desc, ws)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        Wx.copy_(torch.roll(Wx, 1, dims=0))          # new inputs, same buffers
        dH.mul_(-1.0)
        step()
        eager = snapshot()
        for t in (states,) + out:
            t.fill_(float("nan"))
        graph.replay()
        replayed = snapshot()
        api.flashrnn_check(desc, ws)
        for a, r in zip(eager, replayed):
            assert torch.equal(a, r), f"replay {rep} differs from the eager result"


@pytest.mark.parametrize("cell,NH,D,T,B,slices", [(CELL_LSTM, 1, 768, 63, 16, 3), (CELL_GRU, 1, 1024, 70, 16, 3), (CELL_ELMAN, 1, 1536, 157, 15, 5), (CELL_ELMAN, 1, 2048, 9, 15, 1),
                                                  (CELL_LSTM, 3, 272, 18, 15, 2)])
def test_weight_gradient_gemm_with_few_heads(cell, NH, D, T, B, slices):
    """Fewer (head, contraction slice) pairs than XCDs, a number of slices that is no power of two, and a last slice that is
    shorter than the others: the output tiles are dealt out over the XCDs in equal runs."""
    w = Workload(f"fewheads_{cell}_NH{NH}_D{D}", cell, T, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + T)
    # (the slices' partial results are the workspace's largest part, everything else is smaller than one of them)
    assert api.flashrnn_workspace_bytes(api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16)) // (NH * D * w.G * D * 4) == (slices if slices > 1 else 0)
    assert slices == 1 or T * B % ((T * B // slices + 31) // 32 * 32)
    _check(w, with_dlast=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("cell,NH,D,T,B", [(CELL_LSTM, 3, 48, 69, 16), (CELL_GRU, 5, 80, 75, 15), (CELL_ELMAN, 2, 112, 161, 13)])
def test_weight_gradient_gemm_with_heads_that_share_cache_lines(dtype, cell, NH, D, T, B):
    """Heads whose rows are no multiple of 128 bytes with eight and more slices: each XCD takes every eighth slice of all heads."""
    w = Workload(f"shared_{cell}_{dtype}_NH{NH}_D{D}", cell, T, B, NH, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + T)
    assert api.flashrnn_workspace_bytes(api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16 if dtype == "bf16" else api.FLASHRNN_F32)) >= 8 * NH * D * w.G * D * 4
    _check(w, with_dlast=True)


@pytest.mark.parametrize("cell", [CELL_LSTM, CELL_GRU])
@pytest.mark.parametrize("D,bt", [(192, 4), (160, 4), (192, 8), (128, 8), (32, 4), (16, 8)])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 6, 7, 9])
def test_staged_forward_kernels_at_every_pipeline_length(cell, D, bt, T):
    """The staged kernels fetch their inputs up to five steps ahead and park them two ahead: sequences around those distances, a
    ragged last batch tile, contraction lengths that fill the last sparse step of 64 and that leave half of it."""
    w = Workload(f"pipe_{cell}_D{D}_bt{bt}_T{T}", cell, T, bt + 3, 2, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=T + D + bt)
    _check(w, {"FLASHRNN_BT": str(bt)}, with_dlast=True)


@pytest.mark.parametrize("cell", [CELL_LSTM, CELL_GRU, CELL_ELMAN, CELL_GRU4])
@pytest.mark.parametrize("D", [16, 32, 64])
@pytest.mark.parametrize("bt", [4, 8])
def test_staged_forward_kernels_with_an_infinite_state(cell, D, bt):
    """An overflowed h saturates the gates it reaches, with its sign: nothing of it may meet the zero weights behind a contraction of 32."""
    os.environ["FLASHRNN_BT"] = str(bt)
    w = Workload(f"infh_{cell}_D{D}_bt{bt}", cell, 1, bt + 3, 2, D, "bf16", False, bias="uniform0.1", init="uniform0.1", seed=D + bt)
    inp = synth.make_inputs(w)
    inp["states0"][0, 1, 0, 5], inp["states0"][0, w.B - 1, 1, D - 1] = np.inf, -np.inf
    got, ref = pu.run_gpu(w, inp)["states"][1], pu.run_oracle(w, inp)["states"][1]
    fin = np.isfinite(ref)
    assert fin[0, 1, 0].sum() > D // 8      # (a GRU with r = 0 multiplies it by zero itself, and carries the infinite unit on)
    assert np.isfinite(got[fin]).all() and np.abs(got[fin] - ref[fin]).max() <= pu.TOL_BF16_REL * np.abs(ref[fin]).max()


@pytest.mark.parametrize("cell", [CELL_ELMAN, CELL_GRU, CELL_LSTM])
@pytest.mark.parametrize("D", [16, 32, 64])
@pytest.mark.parametrize("bt", [4, 8])
@pytest.mark.parametrize("clip", [None, 0.5])
def test_staged_backward_kernels_with_an_infinite_gradient(cell, D, bt, clip):
    """An overflowed gate gradient: the recurrent term is an infinity with the sign of R, and the clip makes it plus or minus its bound."""
    os.environ["FLASHRNN_BT"] = str(bt)
    w = Workload(f"infdg_{cell}_D{D}_bt{bt}", cell, 2, bt + 3, 2, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D + bt)
    inp = synth.make_inputs(w)
    inp["dH"][1, 1, 0, 5], inp["dH"][1, w.B - 1, 1, D - 1] = np.inf, -np.inf
    got, ref = pu.run_gpu(w, inp, clip=clip), pu.run_oracle(w, inp, clip=clip)
    for k in ("dWx", "dstates0"):
        inf, fin = np.isinf(ref[k]), np.isfinite(ref[k])
        assert np.array_equal(got[k][inf], ref[k][inf])
        assert np.isfinite(got[k][fin]).all() and np.abs(got[k][fin] - ref[k][fin]).max() <= pu.TOL_BF16_REL * np.abs(ref[k][fin]).max()


# ---- the kernels that the planner takes at sizes which the tests above do not ask for: shapes of every contraction length, batch tile and placement

def _small(name, cell, dtype, T, B, NH, D, env, plan=None):
    """One small call pair of a shape; plan = what flashrnn_plan_kernel must say of the forward and the backward call (None: not asked)."""
    w = Workload(f"{name}_{cell}_{dtype}_D{D}_B{B}", cell, T, B, NH, D, dtype, True, bias="uniform0.1", init="uniform0.1", seed=D + B + T)
    os.environ.update(env)
    d = api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16 if dtype == "bf16" else api.FLASHRNN_F32)
    for bwd in (0, 1) if plan else ():
        assert plan[bwd] is None or api.flashrnn_plan_kernel(d, bwd) == plan[bwd], bwd
    _check(w, env, with_dlast=True)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D", [16, 32])
def test_sixteen_row_tiles_with_f32_io_of_the_smallest_heads(cell, D):
    _small("f32_16", cell, "f32", 4, 19, 2, D, {"FLASHRNN_BT": "16"}, ((0, 16, 1),) * 2)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D", [16, 32, 48, 80, 144, 192])
def test_staged_backward_kernels_of_eight_rows(cell, D):
    staged = D < 144 or cell not in (CELL_LSTM, CELL_SLSTM)   # (those spill registers)
    _small("bwd8", cell, "bf16", 5, 11, 2, D, {"FLASHRNN_BT": "8"}, (None, (1, 8, 1) if staged else None))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D,bt", [(16, 8), (80, 4), (80, 8), (128, 4), (128, 8)])
def test_deep_fetch_of_eight_waves_and_of_the_smallest_heads(cell, D, bt):
    _small("deep", cell, "bf16", 9, 11, 2, D, {"FLASHRNN_BT": str(bt), "FLASHRNN_DEEP_FETCH": "2"}, (None, (2, bt, 1)))


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D", [240, 288, 336, 352, 400, 416, 432, 512])
@pytest.mark.parametrize("bt", [4, 8, 16])
@pytest.mark.parametrize("split", ["0", "1"])
def test_split_heads_of_every_contraction_length(cell, D, bt, split):
    """With (1) and without (0) the kernels that have wave roles; two heads, a ragged last tile."""
    _small("lengths", cell, "bf16", 4, bt + 3, 2, D, {"FLASHRNN_BT": str(bt), "FLASHRNN_SPLIT": split})


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D,B,env", [
    (528, 17, {}), (800, 3, {"FLASHRNN_BT": "4"}), (800, 9, {"FLASHRNN_BT": "8"}), (800, 17, {"FLASHRNN_BT": "16"}),
    (1296, 5, {}), (1392, 3, {}), (1408, 3, {}), (1552, 3, {}), (1664, 2, {}), (1792, 13, {}), (2064, 3, {}), (2576, 2, {}),
])
def test_large_heads_of_every_contraction_length(cell, D, B, env):
    """Heads whose blocks of 16 units are no multiple of eight or do not divide among the CUs of an XCD, and members on all XCDs that fetch rows of four."""
    _small("large", cell, "bf16", 2, B, 1, D, env)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D", [256, 352, 416, 512])
@pytest.mark.parametrize("bt", [4, 8, 16])
def test_forward_kernels_of_two_blocks_per_workgroup(cell, D, bt):
    """What batches take whose groups fill the chip: forced onto three groups in rounds of two."""
    env = {"FLASHRNN_BT": str(bt), "FLASHRNN_NWU": "2", "FLASHRNN_GPAR": "2"}
    os.environ.update(env)
    _small("two", cell, "bf16", 5, 2 * bt + 3, 1, D, env)
    assert _with_roles(cell, 5, 2 * bt + 3, 1, D, False) == (8, D // 32)


def _of(fn, *args):
    return pytest.param(fn, args, id="-".join([fn.__name__[5:]] + [str(a) for a in args]))


SPLIT_ENVS = [("bf16", 64, {"FLASHRNN_NWU": "1"}), ("bf16", 64, {"FLASHRNN_NWU": "2"}), ("bf16", 128, {"FLASHRNN_NWU": "2"}), ("bf16", 192, {"FLASHRNN_NWU": "4"}),
              ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 256, {}), ("bf16", 384, {})]


@pytest.mark.parametrize("test,args", [
    _of(t, *a) for t, a in
    [(test_groups_split_over_workgroups, (c, *e)) for c in CELLS for e in SPLIT_ENVS]
    + [(test_recurrent_gradient_clip, (c, clip, "bf16", 128, {"FLASHRNN_MULTI": "1", "FLASHRNN_KS": "4"})) for c in CELLS for clip in (0.0, 0.02)]
    + [(test_split_groups_with_padded_contraction, (c, "bf16", D)) for c in (CELL_LSTM, CELL_GRU, CELL_SLSTM) for D in (208, 320, 640)]
    + [(test_largest_head_takes_a_whole_xcd, ()), (test_backward_groups_take_whole_xcds_and_the_whole_chip_where_they_need_them, ())]
    + [(test_heads_beyond_one_xcd_are_spread_over_the_chip, a) for a in ((CELL_LSTM, 1280, 19, 1), (CELL_SLSTM, 2048, 16, 1), (CELL_ELMAN, 2048, 4, 1), (CELL_GRU4, 1536, 4, 1))]
    + [(test_spread_groups_loop_when_they_do_not_fit, (c,)) for c in CELLS] + [(test_group_loop_when_groups_do_not_fit, (c,)) for c in CELLS]
    + [(test_backward_groups_in_rounds_of_smaller_tiles, a) for a in ((CELL_SLSTM, 8, 256, 66, 4, 2), (CELL_LSTM, 8, 256, 130, 8, 2), (CELL_SLSTM, 1, 768, 65, 8, 24))]
    + [(test_split_groups_on_small_batch_tiles, (c, bt, *e)) for c in CELLS for bt in (8, 4) for e in (("bf16", 256, {}), ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 64, {"FLASHRNN_NWU": "1"}))]
    + [(test_split_groups_pass_every_nan_pattern_on, e) for e in (("bf16", 256, {}), ("bf16", 128, {"FLASHRNN_KS": "4"}), ("bf16", 64, {"FLASHRNN_MULTI": "2", "FLASHRNN_BT": "8"}))]
    + [(test_saturated_gates, (c, init, *e)) for c in CELLS for init in ("uniform0.1_bounded", "zero") for e in (("bf16", 256, {}, 7), ("bf16", 128, {"FLASHRNN_MULTI": "1", "FLASHRNN_KS": "4"}, 18))]
    + [(test_backward_with_recomputed_values, (c, "bf16", 256, 7, 11, {"FLASHRNN_RECOMPUTE_STEPS": "3"})) for c in CELLS]
    + [(test_forward_timeout_survives_the_backward_call, ()), (test_exchange_timeout_is_reported_not_hung, ()), (test_runs_are_bitwise_reproducible, ()),
       (test_forward_backward_replay_from_a_hip_graph, (256,)), (test_large_single_head_split_with_contraction_slices, ())]
])
def test_split_heads_without_wave_roles(test, args):
    """The kernels that exchange h and gate gradients lane by lane run wherever no kernel with wave roles fits (heads of 528, 800, 2576 units, Elman): the
    checks above on them."""
    os.environ["FLASHRNN_SPLIT"] = "0"
    test(*args)


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("D,bt", [(192, 4), (160, 4), (192, 8), (128, 8), (32, 4), (16, 8), (256, 4), (768, 16), (1152, 8)])
def test_one_step_on_the_kernels_of_longer_sequences(cell, D, bt):
    """Calls of one step that do not take the kernel of their own: states carried in place, many heads."""
    env = {"FLASHRNN_STEP": "0"} if D > 1024 else {"FLASHRNN_STEP": "0", "FLASHRNN_BT": str(bt)}
    _small("onestep", cell, "bf16", 1, bt + 3, 2 if D < 512 else 1, D, env)


# (one gate's exchange in Elman; cells whose gates an infinite h saturates)
@pytest.mark.parametrize("cell", [CELL_LSTM, CELL_GRU, CELL_ELMAN, CELL_GRU4])
@pytest.mark.parametrize("NH,D,B,env", [
    (2, 256, 7, {"FLASHRNN_BT": "4"}), (2, 320, 11, {"FLASHRNN_BT": "8"}), (2, 352, 11, {"FLASHRNN_NWU": "2", "FLASHRNN_BT": "8"}), (1, 400, 19, {"FLASHRNN_BT": "16"}),
    (1, 512, 7, {"FLASHRNN_NWU": "2", "FLASHRNN_BT": "4"}), (1, 768, 7, {"FLASHRNN_BT": "4"}), (1, 1024, 11, {"FLASHRNN_BT": "8"}), (1, 1280, 3, {}), (1, 1664, 11, {}),
])
def test_split_heads_with_an_infinite_state(cell, NH, D, B, env):
    """An overflowed h crosses the CUs and saturates the gates it reaches, with its sign: contractions that fill the waves' k-steps and that do not."""
    os.environ.update(env)
    w = Workload(f"infh_{cell}_D{D}_B{B}", cell, 1, B, NH, D, "bf16", False, bias="uniform0.1", init="uniform0.1", seed=D + B)
    inp = synth.make_inputs(w)
    inp["states0"][0, 1, 0, 5], inp["states0"][0, w.B - 1, NH - 1, D - 1] = np.inf, -np.inf
    os.environ["FLASHRNN_STEP"] = "0"
    got, ref = pu.run_gpu(w, inp)["states"][1], pu.run_oracle(w, inp)["states"][1]
    assert _with_roles(cell, 1, w.B, NH, D, 2)[0] == 8
    fin = np.isfinite(ref)
    assert fin[0, 1, 0].sum() > D // 8      # (a GRU with r = 0 multiplies it by zero itself, and carries the infinite unit on)
    assert np.isfinite(got[fin]).all() and np.abs(got[fin] - ref[fin]).max() <= pu.TOL_BF16_REL * np.abs(ref[fin]).max()


@pytest.mark.parametrize("cell", [CELL_ELMAN, CELL_GRU, CELL_LSTM])
@pytest.mark.parametrize("NH,D,env", [
    (2, 256, {"FLASHRNN_BT": "4"}), (1, 320, {"FLASHRNN_BT": "8"}), (2, 208, {"FLASHRNN_BT": "8"}), (1, 640, {"FLASHRNN_BT": "16"}), (1, 896, {"FLASHRNN_BT": "4"}),
    (1, 1024, {"FLASHRNN_BT": "16"}), (1, 1280, {}), (1, 2048, {}),
])
@pytest.mark.parametrize("clip", [None, 0.5])
def test_split_heads_with_an_infinite_gradient(cell, NH, D, env, clip):
    """An overflowed gate gradient: its partial sums are infinities with the sign of R, and the clip makes them plus or minus its bound."""
    os.environ.update(env)
    w = Workload(f"infdg_{cell}_D{D}", cell, 2, 7, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D)
    inp = synth.make_inputs(w)
    inp["Wx"] *= np.float32(0.25)   # (a saved value that rounds to one would make a NaN of the infinity by itself)
    inp["dH"][1, 1, 0, 5], inp["dH"][1, w.B - 1, NH - 1, D - 1] = np.inf, -np.inf
    got, ref = pu.run_gpu(w, inp, clip=clip), pu.run_oracle(w, inp, clip=clip)
    for k in ("dWx", "dstates0"):
        inf, fin = np.isinf(ref[k]), np.isfinite(ref[k])
        # (a GRU's update gate has the sign of h_{t-1} - candidate, and the candidate is saved with eight bits: one unit in some hundred)
        assert np.count_nonzero(got[k][inf] != ref[k][inf]) <= (np.count_nonzero(inf) // 256 if cell == CELL_GRU else 0)
        assert np.isfinite(got[k][fin]).all() and np.abs(got[k][fin] - ref[k][fin]).max() <= pu.TOL_BF16_REL * np.abs(ref[k][fin]).max()


SPLIT_KINDS = [(2, 256, 7, {}), (1, 640, 9, {}), (1, 1024, 5, {}), (1, 1280, 3, {}), (1, 2048, 9, {}), (1, 528, 3, {})]


@pytest.mark.parametrize("cell", CELLS)
@pytest.mark.parametrize("NH,D,B,env", SPLIT_KINDS)
def test_empty_sequences_of_split_heads(cell, NH, D, B, env):
    w = Workload(f"T0_{cell}_D{D}", cell, 0, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D)
    gpu = _check(w, env, with_dlast=True)
    assert np.all(gpu["dR"] == 0) and np.all(gpu["db"] == 0)


@pytest.mark.parametrize("NH,D,B,env", SPLIT_KINDS + [(1, 256, 3, {"FLASHRNN_BT": "4"}), (1, 768, 17, {"FLASHRNN_BT": "16"})])
def test_waits_that_give_up_are_reported_in_both_directions(NH, D, B, env):
    """Every kind of split kernel with waits that give up at once: each direction ends, reports its own timeout, and the next calls are right again."""
    os.environ.update(env)
    w = Workload(f"giveup_D{D}", CELL_SLSTM, 5, B, NH, D, "bf16", True, bias="uniform0.1", init="uniform0.1", seed=D)
    print(f"case {w.name}", flush=True)
    inp = synth.make_inputs(w)
    Wx, R, b, dH = (pu.to_device(inp[k], "bf16") for k in ("Wx", "R", "b", "dH"))
    s0, desc = pu.to_device(inp["states0"], "f32"), api.make_desc(w.cell, w.T, B, NH, D, api.FLASHRNN_BF16)
    states, cache, ws = api.flashrnn_fwd(w.cell, Wx, R, b, s0)
    grads = api.flashrnn_bwd(w.cell, R, b, states, cache, dH, workspace=ws)
    api.flashrnn_check(desc, ws)
    for bwd in (False, True):
        os.environ["FLASHRNN_SPIN_LIMIT"] = "-1"
        if bwd:
            api.flashrnn_bwd(w.cell, R, b, states, cache, dH, workspace=ws)
        else:
            api.flashrnn_fwd(w.cell, Wx, R, b, s0, workspace=ws)
        os.environ["FLASHRNN_SPIN_LIMIT"] = "400000"
        with pytest.raises(api.FlashRNNError) as ei:
            api.flashrnn_check(desc, ws)
        assert ei.value.status == api.FLASHRNN_ERR_TIMEOUT
        again, cache2, _ = api.flashrnn_fwd(w.cell, Wx, R, b, s0, workspace=ws)
        grads2 = api.flashrnn_bwd(w.cell, R, b, again, cache2, dH, workspace=ws)
        api.flashrnn_check(desc, ws)
        assert torch.equal(again, states) and all(torch.equal(x, y) for x, y in zip(grads, grads2))
