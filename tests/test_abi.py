"""CPU-only checks of the boundary: the library loads, exports every symbol the header declares,
and rejects bad descriptors without touching a GPU."""
import ctypes
import os
import re

import pytest

from paper_2412_07752_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "flashrnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(flashrnn_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = api.lib()
    names = _declared_symbols()
    assert set(names) == set(api.EXPORTS), (names, api.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_cell_tables_match_paper_appendix_a():
    assert [api.flashrnn_num_states(c) for c in (0, 1, 2, 3, 4)] == [2, 1, 4, 1, 1]
    assert [api.flashrnn_num_gates(c) for c in (0, 1, 2, 3, 4)] == [4, 3, 4, 1, 4]
    assert api.flashrnn_num_states(7) == -1 and api.flashrnn_num_gates(-1) == -1


def test_status_strings():
    seen = set()
    for s in range(0, -8, -1):
        txt = api.status_string(s)
        assert txt and txt not in seen
        seen.add(txt)
    assert "unknown" in api.status_string(-99)


@pytest.mark.parametrize("bad", [dict(cell=5), dict(T=-1), dict(B=0), dict(NH=0), dict(D=0), dict(io_dtype=3),
                                 dict(recurrent_grad_clip=float("nan"))])
def test_bad_descriptors_are_rejected_on_the_host(bad):
    kw = dict(cell=0, T=4, B=2, NH=1, D=16, io_dtype=api.FLASHRNN_F32)
    kw.update(bad)
    d = api.make_desc(**kw)
    assert api.flashrnn_gate_cache_bytes(d) == 0
    assert api.flashrnn_workspace_bytes(d) == 0
    rc = api.lib().flashrnn_fwd(ctypes.byref(d), None, None, None, None, None, None, None, None)
    assert rc == api.FLASHRNN_ERR_SHAPE
    rc = api.lib().flashrnn_bwd(ctypes.byref(d), *([None] * 12))
    assert rc == api.FLASHRNN_ERR_SHAPE


def test_time_step_slabs_beyond_32_bit_offsets_are_refused():
    """The kernels address one time step of a tensor with 32-bit byte offsets: a shape whose per-step slab reaches 2 GiB
    must be refused, not run with dropped accesses."""
    d = api.make_desc(2, 4, 4096, 64, 1024, api.FLASHRNN_BF16)   # sLSTM states: 4 * 4 B * 2^28 units per step
    assert api.flashrnn_workspace_bytes(d) == 0
    assert api.lib().flashrnn_fwd(ctypes.byref(d), *([None] * 8)) == api.FLASHRNN_ERR_UNSUPPORTED
    d = api.make_desc(2, 4, 64, 64, 1024, api.FLASHRNN_BF16)
    assert api.lib().flashrnn_fwd(ctypes.byref(d), *([None] * 8)) == api.FLASHRNN_ERR_NULL


def test_static_scratch_entry_checks_arguments_first():
    d = api.make_desc(0, 4, 2, 1, 24, api.FLASHRNN_BF16)
    assert api.lib().flashrnn_fwd_static_scratch(ctypes.byref(d), *([None] * 7)) == api.FLASHRNN_ERR_UNSUPPORTED
    assert api.lib().flashrnn_fwd_static_scratch(None, *([None] * 7)) == api.FLASHRNN_ERR_NULL


def test_unsupported_head_size_and_null_pointers():
    d = api.make_desc(0, 4, 2, 1, 24, api.FLASHRNN_BF16)  # D not a multiple of 16
    assert api.lib().flashrnn_fwd(ctypes.byref(d), *([None] * 8)) == api.FLASHRNN_ERR_UNSUPPORTED
    d = api.make_desc(0, 4, 2, 1, 32, api.FLASHRNN_BF16)
    assert api.lib().flashrnn_fwd(ctypes.byref(d), *([None] * 8)) == api.FLASHRNN_ERR_NULL
    assert api.lib().flashrnn_bwd(ctypes.byref(d), *([None] * 12)) == api.FLASHRNN_ERR_NULL
    assert api.lib().flashrnn_fwd(None, *([None] * 8)) == api.FLASHRNN_ERR_NULL
    assert api.lib().flashrnn_check(ctypes.byref(d), None, None) == api.FLASHRNN_OK


def test_sizes_and_plans_of_the_benchmark_configurations():
    from paper_2412_07752_amd import synth
    for w in synth.CONFIGS:
        d = api.make_desc(w.cell, w.T, w.B, w.NH, w.D, api.FLASHRNN_BF16 if w.dtype == "bf16" else api.FLASHRNN_F32)
        slots = {0: 4, 1: 4, 2: 8, 3: 1, 4: 4}[w.cell]   # values saved per (t, row, unit): four, the sLSTM's five padded to eight, Elman one
        assert api.flashrnn_gate_cache_bytes(d) == w.T * w.B * w.NH * w.D * slots * (2 if w.dtype == "bf16" else 4)
        assert api.flashrnn_workspace_bytes(d) > 0
        for bwd in (False, True):
            wgs, per_head, waves = api.flashrnn_plan(d, bwd)
            assert 1 <= wgs <= 256 and waves * 64 <= 1024 and per_head >= 1
    # a head that is too large for the compiled shapes is refused, not mis-run
    d = api.make_desc(0, 4, 2, 1, 4096, api.FLASHRNN_BF16)
    assert api.flashrnn_workspace_bytes(d) == 0
    # ... up to the largest fused head the paper reports (App. H.1) every multiple of 16 has a plan: beyond 1024 units
    # one workgroup per block of 16 units, spread over the whole chip
    for D in (1040, 1536, 2048, 2688):
        d = api.make_desc(0, 4, 16, 1, D, api.FLASHRNN_BF16)
        assert api.flashrnn_workspace_bytes(d) > 0
        for bwd in (False, True):
            assert api.flashrnn_plan(d, bwd)[0] % (D // 16) == 0 and api.flashrnn_plan_kernel(d, bwd)[2] == D // 16
    assert api.flashrnn_workspace_bytes(api.make_desc(0, 4, 2, 1, 2704, api.FLASHRNN_BF16)) == 0


@pytest.mark.parametrize("cell,T,B,NH,D,mode,staged,bt", [
    # more 4-row groups than CUs, one or two waves each: they share a CU, 4-row tiles (with three or four waves 8-row tiles backward)
    (0, 512, 24, 48, 16, 2, 1, 4), (4, 512, 32, 48, 32, 2, 1, 4), (0, 512, 32, 48, 32, 1, 2, 4), (2, 128, 96, 12, 32, 1, 2, 4), (0, 512, 96, 12, 64, 1, 2, 8),
    # ... until the CU is full
    (0, 512, 128, 48, 16, 2, 1, 8), (1, 512, 128, 48, 32, 2, 1, 8),
    # the deep fetch up to 1 MB of saved values per time step
    (0, 512, 64, 48, 32, 1, 2, 4), (0, 512, 85, 48, 32, 1, 1, 4), (2, 512, 32, 48, 32, 1, 2, 4), (2, 512, 64, 48, 32, 1, 1, 4), (0, 512, 200, 12, 16, 1, 2, 4),
])
def test_plans_of_many_small_heads(cell, T, B, NH, D, mode, staged, bt):
    assert api.flashrnn_plan_kernel(api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16), mode) == (staged, bt, 1)


@pytest.mark.parametrize("T,B,NH,D,mode,bt", [
    # more 4-row groups than CUs: one round of 8-row tiles instead of a second one of 4 rows from 80 units on ...
    (64, 96, 12, 80, 0, 8), (64, 96, 12, 96, 2, 8), (64, 96, 12, 128, 2, 8), (64, 170, 12, 96, 2, 4),
    # ... until the memory bounds the call; heads of 48 and 64 units share a CU in 4-row tiles
    (256, 100, 12, 80, 0, 4), (256, 100, 12, 80, 2, 8), (256, 100, 12, 112, 2, 4), (64, 96, 12, 64, 0, 8), (64, 96, 12, 64, 2, 4), (16, 100, 12, 48, 0, 4), (64, 64, 12, 80, 0, 4),
])
def test_forward_plans_of_the_slstm_with_many_groups(T, B, NH, D, mode, bt):
    assert api.flashrnn_plan_kernel(api.make_desc(2, T, B, NH, D, api.FLASHRNN_BF16), mode) == (1, bt, 1)


@pytest.mark.parametrize("cell,D,bt", [(2, 128, 4), (4, 128, 4), (0, 128, 4), (2, 112, 4)])
def test_backward_plans_of_float32_heads_of_128_units(cell, D, bt):
    """Two rounds of 4-row tiles, also of the cells with the most to do per step: 48 steps of 8 x 128 units with 200 rows in 4-row and 8-row tiles, us: sLSTM 296 and 358,
    four-gate GRU 277 and 337, LSTM 295 and 344."""
    assert api.flashrnn_plan_kernel(api.make_desc(cell, 48, 200, 8, D, api.FLASHRNN_F32), True) == (0, bt, 1)


@pytest.mark.parametrize("cell,NH,D,B,step", [
    # one-step calls: a kernel of their own, but where its batch tiles read R so often that the persistent kernels are faster
    (2, 4, 192, 1, True), (2, 4, 192, 16, True), (2, 24, 192, 4, True), (2, 24, 192, 32, False), (2, 32, 192, 2, False), (0, 12, 512, 8, True), (0, 12, 512, 16, False),
    (0, 4, 1024, 8, True), (2, 4, 1024, 64, False), (2, 64, 128, 1, True), (2, 96, 128, 1, False), (1, 64, 80, 2, True), (1, 64, 80, 16, False),
    (3, 24, 128, 2, True), (3, 24, 128, 8, False), (3, 24, 384, 8, True), (3, 24, 384, 12, False), (3, 96, 64, 2, False),
])
def test_one_step_plans_of_many_heads_and_rows(cell, NH, D, B, step):
    d = api.make_desc(cell, 1, B, NH, D, api.FLASHRNN_BF16)
    for mode in (0, 2):
        staged, rows, split = api.flashrnn_plan_kernel(d, mode)
        assert (staged == 1 and split == D // 16 and rows == (1 if B == 1 else 4)) == step


def test_weight_gradients_of_very_wide_layers_keep_64_bit_offsets():
    """The weight-gradient kernel of the largest tile reaches the 32 rows of a round with offsets below 2^31: the library takes it only where the last byte of the last
    row is in reach, and a call may be far wider than that (one batch row: up to 2^30 gate columns)."""
    in_reach = getattr(api.lib(), "_ZN8flashrnn18dr_square_in_reachEiiib")
    in_reach.restype = ctypes.c_bool
    for G in (1, 4):
        for D in (208, 256, 1024):
            edge = (1 << 31) // (32 * 2 * G * D)
            for NH in (1, 8, edge - 1, edge, edge + 1, 2 * edge, 4 * edge, 31 * edge):
                assert in_reach(NH, D, G, False) == (32 * 2 * G * NH * D < 1 << 31), (NH, D, G)
                assert not in_reach(NH, D, G, True)
    # LSTM, 40000 heads of 256 units, one row: an accepted call whose rounds span 2.6 GB
    assert api.flashrnn_workspace_bytes(api.make_desc(0, 32, 1, 40000, 256, api.FLASHRNN_BF16)) > 0
    assert not in_reach(40000, 256, 4, False)


@pytest.mark.parametrize("cell,T,B,NH,D,dtype", [(2, 40, 192, 8, 256, api.FLASHRNN_BF16), (2, 1024, 16, 3, 256, api.FLASHRNN_BF16), (0, 333, 11, 3, 80, api.FLASHRNN_BF16), (1, 1000, 64, 8, 128, api.FLASHRNN_BF16),
                                                 (4, 77, 200, 16, 112, api.FLASHRNN_F32), (3, 2048, 128, 16, 128, api.FLASHRNN_BF16), (2, 7, 1000, 8, 1024, api.FLASHRNN_BF16), (0, 1, 3, 1, 16, api.FLASHRNN_F32),
                                                 (2, 0, 16, 4, 192, api.FLASHRNN_BF16)])
def test_windows_of_the_recomputing_backward_pass_stay_within_their_limit(cell, T, B, NH, D, dtype):
    """The records of a window take 80 MiB at most, or one step's where that is more; and no more windows than that takes."""
    d = api.make_desc(cell, T, B, NH, D, dtype)
    up = lambda n: (n + 255) // 256 * 256
    slots = {0: 4, 1: 4, 2: 8, 3: 1, 4: 4}[cell]
    step = B * NH * D * slots * (4 if dtype == api.FLASHRNN_F32 else 2)
    records = api.lib().flashrnn_recompute_workspace_bytes(ctypes.byref(d)) - api.flashrnn_workspace_bytes(d) - 2 * up(api.flashrnn_num_states(cell) * B * NH * D * 4)
    assert records <= up(max(80 << 20, step))
    windows = max(1, -(-T // max(1, (80 << 20) // step)))
    assert records == up(max(1, -(-T // windows)) * step)
