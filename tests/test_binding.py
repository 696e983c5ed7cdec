"""CPU-only checks of what the Python binding hands to the library: a stand-in for the library records the descriptors."""
import numpy as np
import pytest
import torch

from paper_2412_07752_amd import api, build


class _Library:
    """Answers like the real library, but records what a compute call gets instead of launching anything."""

    def __init__(self):
        self.real, self.seen = api.lib(), []

    def __getattr__(self, name):
        if name not in ("flashrnn_fwd", "flashrnn_fwd_static_scratch", "flashrnn_bwd", "flashrnn_bwd_recompute"):
            return getattr(self.real, name)

        def call(desc, *args):
            self.seen.append((name, desc._obj.cell, desc._obj.recurrent_grad_clip))
            return api.FLASHRNN_OK
        return call


@pytest.fixture
def library(monkeypatch):
    rec = _Library()
    monkeypatch.setattr(api, "lib", lambda: rec)
    monkeypatch.setattr(api, "_chk", lambda *a, **k: None)   # (host tensors)
    monkeypatch.setattr(api, "_stream", lambda stream: None)
    return rec


@pytest.mark.parametrize("recompute", [False, True])
@pytest.mark.parametrize("holder", [lambda: torch.tensor(1.0), lambda: np.array(1.0), lambda: torch.ones(1, dtype=torch.float64)])
def test_the_clip_is_read_at_every_call(library, holder, recompute):
    """A clip that the caller keeps in a tensor or an array and changes in place between calls."""
    T, B, G, NH, D = 2, 1, 4, 1, 16
    dH, Wx, R, b = torch.zeros(T, B, NH, D), torch.zeros(T, B, G, NH, D), torch.zeros(NH, D, G, D), torch.zeros(NH, G, D)
    states, cache, ws = torch.zeros(T + 1, 2, B, NH, D), torch.zeros(1 << 12, dtype=torch.uint8), torch.zeros(1)
    clip = holder()
    for value in (1.0, 2.0, 0.5, -1.0, 0.0):
        clip[...] = value
        if recompute:
            api.flashrnn_bwd_recompute(api.FLASHRNN_LSTM, Wx, R, b, states, dH, workspace=ws, recurrent_grad_clip=clip)
        else:
            api.flashrnn_bwd(api.FLASHRNN_LSTM, R, b, states, cache, dH, workspace=ws, recurrent_grad_clip=clip)
        assert library.seen[-1][2] == value


def test_cells_given_as_arrays_or_tensors(library):
    """Whatever int() takes names a cell, in the tables and in the calls."""
    Wx, R, b, ws = torch.zeros(2, 1, 3, 1, 16), torch.zeros(1, 16, 3, 16), torch.zeros(1, 3, 16), torch.zeros(1)
    cell = torch.tensor(api.FLASHRNN_LSTM)
    for c in (cell, np.array(api.FLASHRNN_LSTM), np.int64(api.FLASHRNN_LSTM), True - 1):
        assert (api.flashrnn_num_states(c), api.flashrnn_num_gates(c)) == (2, 4)
    cell.fill_(api.FLASHRNN_GRU)
    assert (api.flashrnn_num_states(cell), api.flashrnn_num_gates(cell)) == (1, 3)
    for c in (cell, np.array(api.FLASHRNN_GRU)):
        api.flashrnn_fwd(c, Wx, R, b, save_for_backward=False, workspace=ws)
        api.flashrnn_fwd_static_scratch(c, Wx, R, b, save_for_backward=False)
        assert [s[1] for s in library.seen[-2:]] == [api.FLASHRNN_GRU] * 2


def _call(T=1, B=2, cell=None, dev="cpu", dtype=torch.bfloat16):
    cell = api.FLASHRNN_LSTM if cell is None else cell
    G, S, NH, D = 4, 2, 1, 16
    rng = torch.Generator().manual_seed(3)
    r = lambda *s: torch.randn(s, generator=rng).to(dtype).to(dev)
    return dict(cell=cell, Wx=r(T, B, G, NH, D), R=r(NH, D, G, D), b=r(NH, G, D), states0=torch.randn((S, B, NH, D), generator=rng).to(dev),
                save_for_backward=False, workspace=None, states=torch.zeros((T + 1, S, B, NH, D), device=dev), gate_cache=None)


@pytest.mark.parametrize("built_for", [None, "python 3.10, torch 2.9.1 0000", ""])
def test_a_native_module_of_another_torch_or_python_is_not_bound(built_for, monkeypatch):
    """It would read tensors through a layout that need not be theirs; that it loads says nothing."""
    import sys
    import types
    import paper_2412_07752_amd as package
    module = types.ModuleType("paper_2412_07752_amd._flashrnn_binding")
    if built_for is not None:
        module.built_for = built_for
    monkeypatch.setitem(sys.modules, module.__name__, module)
    monkeypatch.setattr(package, "_flashrnn_binding", module, raising=False)
    with pytest.warns(RuntimeWarning, match="built for"):
        assert api._load_native() is None
    module.built_for = build.binding_stamp()
    assert api._load_native() is module


def test_a_missing_native_module_is_told_of(monkeypatch):
    import sys
    import paper_2412_07752_amd as package
    monkeypatch.setitem(sys.modules, "paper_2412_07752_amd._flashrnn_binding", None)
    monkeypatch.delattr(package, "_flashrnn_binding", raising=False)
    with pytest.warns(RuntimeWarning, match="native binding"):
        assert api._load_native() is None


def test_native_calls_hand_back_host_tensors():
    """Nothing but device tensors is the native module's business."""
    api.lib()
    if api._native is None:
        pytest.skip("the native module was built against another torch")
    a = _call()
    assert api._native.fwd(*a.values()) == 1
    assert api._native.fwd(*dict(a, states0=None).values()) == 1
    assert api._native.fwd(1, 2) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_native_calls_take_what_is_plain_and_hand_back_the_rest(dtype):
    """Plain calls are made, not handed back; every single change to one is handed back (or, for a pointer that the library refuses, comes back as its status)."""
    api.lib()
    assert api._native is not None
    desc = api.make_desc(api.FLASHRNN_LSTM, 3, 2, 1, 16, api.FLASHRNN_BF16 if dtype is torch.bfloat16 else api.FLASHRNN_F32)
    ws, cache = api.alloc_workspace(desc, "cuda"), torch.zeros(api.flashrnn_gate_cache_bytes(desc), dtype=torch.uint8, device="cuda")
    a = dict(_call(T=3, dev="cuda", dtype=dtype), workspace=ws)
    native = lambda **change: api._native.fwd(*dict(a, **change).values())
    for plain in ({}, {"workspace": None}, {"states0": None}, {"save_for_backward": True, "gate_cache": cache}, {"gate_cache": cache}, {"Wx": torch.nn.Parameter(a["Wx"])}):
        assert native(**plain) == api.FLASHRNN_OK
    strided = lambda t: t.transpose(0, -1).contiguous().transpose(0, -1)
    other = torch.float32 if dtype is torch.bfloat16 else torch.bfloat16
    changes = [("cell", c) for c in (0.0, np.int64(0), True, -1, 5, 99, 10 ** 30, api.FLASHRNN_GRU)]
    changes += [("save_for_backward", v) for v in (1, None, np.bool_(False))] + [("states", None), ("Wx", None), ("R", None), ("b", None)]
    changes += [("Wx", np.zeros(3)), ("Wx", a["Wx"][0]), ("Wx", a["Wx"][:, :, :3].contiguous()), ("Wx", a["Wx"][:2].contiguous())]
    changes += [("R", a["R"][:, :, :, :8].contiguous()), ("b", a["b"][:, :2].contiguous()), ("states", a["states"][:3]), ("states0", a["states0"][:, :1].contiguous())]
    for name in ("Wx", "R", "b", "states0", "states"):
        changes += [(name, a[name].cpu()), (name, a[name].double())]
        if name in ("Wx", "R", "b"):
            changes.append((name, a[name].to(other)))
    changes += [(name, strided(a[name])) for name in ("R", "states0", "states")] + [("Wx", a["Wx"].transpose(0, 1).contiguous().transpose(0, 1))]
    changes += [("workspace", ws.cpu()), ("workspace", 0), ("states0", 0.0)]
    for name, value in changes:
        assert native(**{name: value}) == 1, (name, value)
    assert native(save_for_backward=True) == 1 and native(save_for_backward=True, gate_cache=cache.cpu()) == 1
    assert native(workspace=ws[1:]) == api.FLASHRNN_ERR_WORKSPACE
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("native", [True, False])
def test_calls_run_on_the_current_stream(native, static, monkeypatch):
    """Inputs that another stream is still to write, behind a wait: a call made while that stream is the current one sees them."""
    api.lib()
    if not native:
        monkeypatch.setattr(api, "_native", None)
    desc = api.make_desc(api.FLASHRNN_LSTM, 3, 2, 1, 16, api.FLASHRNN_BF16)
    a = _call(T=3, dev="cuda")
    a.pop("workspace")
    kw = {} if static else dict(workspace=api.alloc_workspace(desc, "cuda"))
    fn = api.flashrnn_fwd_static_scratch if static else api.flashrnn_fwd
    want = fn(**a, **kw)[0].clone()
    late, stream = a["Wx"].clone(), torch.cuda.Stream()
    a["Wx"].zero_()
    a["states"].zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(20_000_000)   # (clocks: ten milliseconds)
        a["Wx"].copy_(late)
        fn(**a, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a["states"], want)


@pytest.mark.gpu
def test_native_calls_and_calls_through_python_are_the_same(monkeypatch):
    """The same buffers, results and refusals with and without the native module, for every argument that it hands back."""
    api.lib()
    assert api._native is not None
    desc = api.make_desc(api.FLASHRNN_LSTM, 3, 2, 1, 16, api.FLASHRNN_BF16)
    results = {}
    for native in (True, False):
        if not native:
            monkeypatch.setattr(api, "_native", None)
        a = _call(T=3, dev="cuda")
        a.pop("workspace")
        ws, cache = api.alloc_workspace(desc, "cuda"), torch.zeros(api.flashrnn_gate_cache_bytes(desc), dtype=torch.uint8, device="cuda")
        out = []
        for change in ({}, {"states0": None}, {"states": None}, {"save_for_backward": True}, {"save_for_backward": True, "gate_cache": cache},
                       {"Wx": a["Wx"].transpose(0, 1).contiguous().transpose(0, 1)}, {"Wx": a["Wx"][:, :, :3].contiguous()}, {"R": a["R"].float()}, {"R": a["R"].cpu()},
                       {"b": a["b"][:, :2]}, {"states0": a["states0"].bfloat16()}, {"states": a["states"][:2]}, {"cell": 7}, {"Wx": torch.nn.Parameter(a["Wx"])},
                       {"R": a["R"].reshape(-1)[1:], }):
            for kw in (dict(workspace=ws), dict()):
                fn = api.flashrnn_fwd if kw else api.flashrnn_fwd_static_scratch
                args = dict(a, **kw)
                args.update(change)
                if args.get("states") is not None:
                    args["states"].zero_()
                try:
                    res = fn(**args)
                    torch.cuda.synchronize()
                    out.append([x.clone().cpu() if i < 2 and x is not None else x is None for i, x in enumerate(res)])
                except Exception as e:
                    out.append((type(e).__name__, str(e)))
        results[native] = out
    assert len(results[True]) == len(results[False])
    for x, y in zip(results[True], results[False]):
        assert type(x) is type(y)
        if isinstance(x, tuple):
            assert x == y
        else:
            assert all(torch.equal(p, q) if torch.is_tensor(p) else p == q for p, q in zip(x, y))
