"""dR of the largest output tile (256 x 256, heads of more than 192 units with many tiles) against 64-bit sums over the same gate gradients and states: contraction lengths
around a round of 32 rows and its double, ragged slices, units and gate columns that do not fill a tile.

Bound: products of bf16 values are exact in float32; T B of them are added in chains and slices: 2^-24 sqrt(T B) of the root of the summed squares, times 4."""
import numpy as np
import pytest
import torch

from paper_2412_07752_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell,NH,D", [(api.FLASHRNN_LSTM, 8, 256), (api.FLASHRNN_SLSTM, 4, 480), (api.FLASHRNN_ELMAN, 8, 1024), (api.FLASHRNN_GRU, 11, 256), (api.FLASHRNN_GRU4, 8, 496)])
@pytest.mark.parametrize("T,B", [(1, 1), (1, 31), (2, 16), (3, 11), (1, 64), (13, 5), (7, 37), (40, 33)])
def test_weight_gradient_of_the_largest_tile(cell, NH, D, T, B):
    G, S = api.flashrnn_num_gates(cell), api.flashrnn_num_states(cell)
    gen = torch.Generator(device="cuda").manual_seed(T * 100 + B)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    Wx, R, b, dH = rnd(T, B, G, NH, D), rnd(NH, D, G, D) * D ** -0.5, rnd(NH, G, D) * 0.1, rnd(T, B, NH, D)
    s0 = torch.rand((S, B, NH, D), generator=gen, device="cuda") * 0.5 + (1.0 if cell == api.FLASHRNN_SLSTM else 0.0)
    if S == 4:
        s0[1] *= 0.5
        s0[3] = 0.0
    desc = api.make_desc(cell, T, B, NH, D, api.FLASHRNN_BF16)
    states, cache, ws = api.flashrnn_fwd(cell, Wx, R, b, s0)
    dR = torch.full((NH, D, G, D), float("nan"), device="cuda")
    out = (torch.empty((T, B, G, NH, D), dtype=torch.bfloat16, device="cuda"), dR, torch.empty((NH, G, D), device="cuda"), torch.empty((S, B, NH, D), device="cuda"))
    dWx = api.flashrnn_bwd(cell, R, b, states, cache, dH, workspace=ws, out=out)[0]
    api.flashrnn_check(desc, ws)
    h = states[:-1, 0].bfloat16().double().reshape(T * B, NH, D)
    dg = dWx.double().reshape(T * B, G, NH, D)
    gates = [g for g in range(G) if not (cell == api.FLASHRNN_GRU and g == 2)]   # (the recurrent-side gradient of the GRU's candidate is not an output)
    for n in range(0, NH, 3):
        ref = torch.stack([h[:, n].t().contiguous() @ dg[:, g, n] for g in gates], dim=1)
        size = torch.stack([(h[:, n] ** 2).t().contiguous() @ (dg[:, g, n] ** 2) for g in gates], dim=1).sqrt()
        got = dR[n][:, gates].double()
        bound = 4 * 2.0 ** -24 * np.sqrt(T * B) * size + 1e-30
        assert bool((abs(got - ref) <= bound + 2.0 ** -24 * abs(ref)).all()), f"head {n}: {float((abs(got - ref) / bound).max()):.2f} of the bound"
