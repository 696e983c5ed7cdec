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


def _records(cell, Wx, states0):
    """The values that one step saves for the backward pass [n, values]: every gate by itself, in float64."""
    n, G = Wx.shape
    B = n // 16
    wx = torch.from_numpy(np.ascontiguousarray(Wx.reshape(B, 16, G).transpose(0, 2, 1))[None, :, :, None, :]).cuda()
    s0 = torch.from_numpy(np.ascontiguousarray(states0.reshape(-1, B, 1, 16))).cuda()
    R, b = torch.zeros((1, 16, G, 16), device="cuda"), torch.zeros((1, G, 16), device="cuda")
    states, cache, _ = api.flashrnn_fwd(cell, wx.contiguous(), R, b, s0)
    torch.cuda.synchronize()
    return cache.view(torch.float32).reshape(n, -1).cpu().numpy().astype(np.float64), states[1].reshape(-1, n).cpu().numpy().astype(np.float64)


def _off(got, ref):
    """Root mean square of the relative error, in roundings."""
    return np.sqrt(np.mean(((got - ref) / ref) ** 2)) / ULP


@pytest.mark.parametrize("reach", [0.1, 0.6, 2.0, 5.0, 20.0, 80.0])
def test_sigmoids_are_no_further_off_than_the_plain_formula(reach):
    """1 / (1 + e^-x) with each of its three steps correctly rounded; two hundredths for the sample."""
    x = np.random.default_rng(3).uniform(-reach, reach, 1 << 16).astype(np.float32)
    ones = np.ones((4, x.size), np.float32)
    lstm, _ = _records(api.FLASHRNN_LSTM, np.stack([x] * 4, axis=1), ones[:2])
    slstm, _ = _records(api.FLASHRNN_SLSTM, np.stack([np.zeros_like(x), -x, x, x], axis=1), ones)
    ref = _sig(x.astype(np.float64))
    plain = (np.float32(1) / (np.float32(1) + np.exp(-x.astype(np.float64)).astype(np.float32))).astype(np.float64)
    for got in (lstm[:, 0], lstm[:, 1], lstm[:, 3], slstm[:, 3], slstm[:, 4]):   # (the sLSTM's last: sig(-f), f = -x)
        assert _off(got, ref) <= 1.02 * _off(plain, ref)


def test_saturated_gates_are_zero_or_one():
    """Beyond the reach of float32 a gate is exactly open or shut, as in 1 / (1 + e^-x), and what is masked by an infinite pre-activation is gone."""
    far = np.float32([105.0, 110.0, 111.0, 200.0, 1e4, 1e30, 3e38, np.inf] * 2)
    ones = np.ones((4, far.size), np.float32)
    for x, want in ((far, 1.0), (-far, 0.0)):
        lstm, _ = _records(api.FLASHRNN_LSTM, np.stack([x] * 4, axis=1), ones[:2])
        assert (lstm[:, [0, 1, 3]] == want).all()
        gru, _ = _records(api.FLASHRNN_GRU, np.stack([x] * 3, axis=1), ones[:1])
        assert (gru[:, :2] == want).all()
    zeros = np.zeros_like(far)
    slstm, states = _records(api.FLASHRNN_SLSTM, np.stack([zeros - 5, far, zeros, far], axis=1), np.stack([zeros, zeros + 1, zeros + 1, zeros]))
    assert (slstm[:, 3] == 1).all() and (slstm[:, 4] == 0).all()   # output gate; what the forget gate still lacks
    assert (states[3] == 0).all()                                  # m = log sig(f) + m0
    # below the smallest normal number: what is left of it, to half a unit of the last place there is
    x = np.linspace(-103.0, -86.0, 1024).astype(np.float32)
    lstm, _ = _records(api.FLASHRNN_LSTM, np.stack([x] * 4, axis=1), np.ones((2, x.size), np.float32))
    ref = _sig(x.astype(np.float64))
    assert np.all(np.abs(lstm[:, 3] - ref) <= 3 * ULP * ref + 1.5 * 2.0 ** -149)


@pytest.mark.parametrize("reach", [0.1, 0.6, 2.0, 5.0, 20.0, 80.0])
def test_log_sigmoids_and_exponentials_are_no_further_off_than_the_plain_formulas(reach):
    """min(x, 0) - log(1 + e^-|x|) and e^x with each step correctly rounded, but for the exponential: on the hardware's 2^f the library's comes to 1.02 to 1.04 times the error
    of correct rounding (two roundings of the exponent's fraction instead of one: 1.06), which log sig(x) -> -e^-x takes over; half a hundredth for the sample."""
    x = np.random.default_rng(4).uniform(-reach, reach, 1 << 16).astype(np.float32)
    zeros = np.zeros_like(x)
    # m = max(log sig(f) + m0, i) with m0 = 0 and i far below
    _, states = _records(api.FLASHRNN_SLSTM, np.stack([zeros - 1000, x, zeros, zeros], axis=1), np.stack([zeros, zeros, zeros + 1, zeros]))
    xd = x.astype(np.float64)
    ref = np.minimum(xd, 0) - np.log1p(np.exp(-np.abs(xd)))
    log1p = np.log1p(np.exp(-np.abs(xd)).astype(np.float32).astype(np.float64)).astype(np.float32)
    plain = (np.minimum(x, np.float32(0)) - log1p).astype(np.float64)
    assert _off(states[3], ref) <= 1.045 * _off(plain, ref)
    # weights e^(a - m), e^(i - m): f = 1000 (log sig = 0), m0 = 0 and i = +-x
    for sign in (1, -1):
        i = sign * x
        rec, _ = _records(api.FLASHRNN_SLSTM, np.stack([i, zeros + 1000, zeros, zeros], axis=1), np.stack([zeros, zeros, zeros + 1, zeros]))
        m = np.maximum(i, 0).astype(np.float64)
        for got, arg in ((rec[:, 0], i - m), (rec[:, 1], -m)):
            some = arg != 0
            assert (got[~some] == 1).all()
            e = np.exp(arg[some])
            assert _off(got[some], e) <= 1.045 * _off(e.astype(np.float32).astype(np.float64), e)
