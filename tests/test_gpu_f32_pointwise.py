"""The float32 point-wise functions (sigmoid, tanh, log sigmoid, exponentials), argument by argument, through the C ABI: one time step with R = 0 and b = 0 is a function of Wx and
the initial states alone.  Arguments cover the places where the formulas change or saturate.

Bound: a handful of float32 roundings (2^-24 each) of every intermediate value: 3 for a sigmoid or a tanh, 5 for log sigmoid, and the exact arithmetic's own roundings
on top -- 8 roundings of the largest term that enters a state."""
import numpy as np
import pytest
import torch

from paper_2412_07752_amd import api

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24
EDGES = [0.0, 1e-30, 1e-8, 1e-3, 0.3, 0.6249, 0.625, 0.6251, 0.9, 1.0, 2.0, 5.0, 9.0, 17.0, 19.9, 20.1, 43.0, 86.9, 87.1, 87.9, 88.1, 89.0, 103.0, 105.0, 120.0, 1e4, 1e30]


def _arguments(n):
    rng = np.random.default_rng(7)
    x = np.concatenate([EDGES, -np.array(EDGES), rng.normal(0, 1, n // 2), rng.uniform(-25, 25, n)])[:n]
    return x.astype(np.float32)


def _step(cell, Wx, states0):
    """One step of NH = 1, D = 16 from columns Wx[n, G], states0[S, n] (n a multiple of 16): states after it [S, n] in float64."""
    n, G = Wx.shape
    B = n // 16
    wx = torch.from_numpy(np.ascontiguousarray(Wx.reshape(B, 16, G).transpose(0, 2, 1))[None, :, :, None, :]).cuda()
    s0 = torch.from_numpy(np.ascontiguousarray(states0.reshape(-1, B, 1, 16))).cuda()
    R, b = torch.zeros((1, 16, G, 16), device="cuda"), torch.zeros((1, G, 16), device="cuda")
    states, _, _ = api.flashrnn_fwd(cell, wx.contiguous(), R, b, s0, save_for_backward=False)
    torch.cuda.synchronize()
    return states[1].reshape(-1, n).cpu().numpy().astype(np.float64)


def _sig(x):
    return np.where(x >= 0, 1 / (1 + np.exp(-np.abs(x))), np.exp(-np.abs(x)) / (1 + np.exp(-np.abs(x))))


@pytest.mark.parametrize("rows", [3, 40])   # (4-row tiles; 16-row tiles take over from four workgroups per CU on, forced below)
@pytest.mark.parametrize("bt", [None, "8", "16"])
def test_elman_is_tanh(rows, bt, monkeypatch):
    if bt:
        monkeypatch.setenv("FLASHRNN_BT", bt)
    x = _arguments(16 * rows)
    h = _step(api.FLASHRNN_ELMAN, x[:, None], np.zeros((1, x.size), np.float32))[0]
    ref = np.tanh(x.astype(np.float64))
    assert np.all(np.abs(h - ref) <= 3 * ULP * np.abs(ref) + 1e-40)


@pytest.mark.parametrize("bt", ["4", "16"])
def test_lstm_gates(bt, monkeypatch):
    monkeypatch.setenv("FLASHRNN_BT", bt)
    x = _arguments(640)
    y = x[::-1].copy()
    Wx = np.stack([x, y, np.roll(x, 3), np.roll(y, 5)], axis=1)
    c0 = np.random.default_rng(1).normal(0, 1, x.size).astype(np.float32)
    h, c = _step(api.FLASHRNN_LSTM, Wx, np.stack([np.zeros_like(c0), c0]))
    w = Wx.astype(np.float64)
    i, f, z, o = _sig(w[:, 0]), _sig(w[:, 1]), np.tanh(w[:, 2]), _sig(w[:, 3])
    c_ref = f * c0 + i * z
    assert np.all(np.abs(c - c_ref) <= 8 * ULP * (np.abs(f * c0) + np.abs(i * z)) + 1e-37)
    h_ref = o * np.tanh(c)
    assert np.all(np.abs(h - h_ref) <= 8 * ULP * np.abs(h_ref) + 1e-37)


@pytest.mark.parametrize("bt", ["4", "16"])
def test_slstm_gates(bt, monkeypatch):
    monkeypatch.setenv("FLASHRNN_BT", bt)
    x = np.clip(_arguments(640), -300, 300)
    Wx = np.stack([np.abs(x[::-1]) % 30, x, np.roll(x, 3), np.roll(x, 5)], axis=1).astype(np.float32)
    rng = np.random.default_rng(2)
    n0 = rng.uniform(0.5, 1.5, x.size).astype(np.float32)
    c0 = (n0 * rng.uniform(-1, 1, x.size)).astype(np.float32)
    m0 = rng.uniform(-2, 2, x.size).astype(np.float32)
    h, c, n, m = _step(api.FLASHRNN_SLSTM, Wx, np.stack([np.zeros_like(c0), c0, n0, m0]))
    w = Wx.astype(np.float64)
    lf = np.minimum(w[:, 1], 0) - np.log1p(np.exp(-np.abs(w[:, 1])))
    a = lf + m0
    m_ref = np.maximum(a, w[:, 0])
    assert np.all(np.abs(m - m_ref) <= 6 * ULP * (np.abs(lf) + np.abs(m0) + np.abs(m_ref)))
    # the weights are exponentials of differences: an error of one rounding of m or log sig(f) + m is a relative error of theirs
    rel = 8 * ULP * (1 + np.abs(lf) + np.abs(m0) + np.abs(m_ref))
    fg, ig = np.exp(a - m_ref), np.exp(w[:, 0] - m_ref)
    z = np.tanh(w[:, 2])
    assert np.all(np.abs(n - (fg * n0 + ig)) <= rel * (fg * n0 + ig) + 1e-37)
    assert np.all(np.abs(c - (fg * c0 + ig * z)) <= rel * (fg * np.abs(c0) + ig * np.abs(z)) + 1e-37)
    h_ref = _sig(w[:, 3]) * c / n
    assert np.all(np.abs(h - h_ref) <= 8 * ULP * np.abs(h_ref) + 1e-37)


@pytest.mark.parametrize("cell", [api.FLASHRNN_ELMAN, api.FLASHRNN_LSTM, api.FLASHRNN_SLSTM])
def test_nan_and_infinities(cell):
    """A NaN in any gate is a NaN in h; infinite pre-activations saturate."""
    G, S = api.flashrnn_num_gates(cell), api.flashrnn_num_states(cell)
    s0 = np.ones((S, 16), np.float32)
    for g in range(G):
        Wx = np.full((16, G), 0.5, np.float32)
        Wx[3, g] = np.nan
        h = _step(cell, Wx, s0)[0]
        assert np.isnan(h[3]) and np.isfinite(np.delete(h, 3)).all()
    Wx = np.full((16, G), 0.5, np.float32)
    Wx[2, -1], Wx[5, -1] = np.inf, -np.inf   # the output gate, Elman's only one
    h = _step(cell, Wx, s0)[0]
    base = _step(cell, np.full((16, G), 0.5, np.float32), s0)[0][0]
    if cell == api.FLASHRNN_ELMAN:
        assert h[2] == 1.0 and h[5] == -1.0
    else:
        assert abs(h[5]) < 1e-30 and abs(h[2] * float(_sig(np.float64(0.5))) - base) < 1e-5 * abs(base)
