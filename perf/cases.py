"""The cases this framework's speed is measured on.

Each case is one use of the public entry points of paper_2412_07752_amd.api, as bench.py and a user's program make it: buffers
allocated once, then one call (or pair of calls) per pass on the current stream.

mode  "infer"      flashrnn_fwd that saves nothing
      "train"      flashrnn_fwd + flashrnn_bwd
      "recompute"  flashrnn_fwd that saves nothing + flashrnn_bwd_recompute
      "decode"     T calls of flashrnn_fwd_static_scratch with one time step each, the states carried from call to call
clip  bound of the recurrent gradient term per value (0: off);  init  the caller passes initial states (else zeros);
last  the caller passes gradients of the last states.
"""
import ctypes
import math

import torch

from paper_2412_07752_amd import api

CELLS = {"lstm": api.FLASHRNN_LSTM, "gru": api.FLASHRNN_GRU, "slstm": api.FLASHRNN_SLSTM, "elman": api.FLASHRNN_ELMAN, "gru4": api.FLASHRNN_GRU4}
GATES = {"lstm": 4, "gru": 3, "slstm": 4, "elman": 1, "gru4": 4}
STATES = {"lstm": 2, "gru": 1, "slstm": 4, "elman": 1, "gru4": 1}
FORGET = 1   # index of the forget gate of LSTM and sLSTM


def _case(name, mode, cell, dtype, T, B, NH, D, init=False, last=False, clip=0.0):
    return {"name": name, "mode": mode, "cell": cell, "dtype": dtype, "T": T, "B": B, "NH": NH, "D": D, "init": init, "last": last, "clip": clip}


def listed():
    return [
        # the smallest call: a short float32 sequence through one small head (latency, launches)
        _case("lstm_f32_infer_1x64_b4_t32", "infer", "lstm", "f32", 32, 4, 1, 64),
        # token-by-token generation: one time step per call, one sequence, states carried by the caller
        _case("slstm_decode_4x192_b1_t16", "decode", "slstm", "bf16", 16, 1, 4, 192, init=True),
        # float32 training on ragged sizes (gradient checks, small models)
        _case("gru_f32_train_4x96_b12_t150", "train", "gru", "f32", 150, 12, 4, 96, init=True),
        # bf16 training, odd everything, with the options of the backward call in use
        _case("lstm_train_3x80_b11_t333", "train", "lstm", "bf16", 333, 11, 3, 80, init=True, last=True, clip=1.0),
        # the benchmark's default workload: one sLSTM layer of 768 units in four heads
        _case("slstm_train_4x192_b16_t256", "train", "slstm", "bf16", 256, 16, 4, 192),
        # the usual language-model layer: twelve small heads, context 1024
        _case("lstm_train_12x64_b16_t1024", "train", "lstm", "bf16", 1024, 16, 12, 64),
        # many short steps at once: half of the chip streams
        _case("gru_train_8x128_b64_t512", "train", "gru", "bf16", 512, 64, 8, 128),
        # one head over the whole layer, inference on a batch (prefill)
        _case("lstm_infer_1x768_b16_t1024", "infer", "lstm", "bf16", 1024, 16, 1, 768),
        # memory-saving training: the saved values are formed again in the backward pass
        _case("slstm_recompute_3x256_b16_t1024", "recompute", "slstm", "bf16", 1024, 16, 3, 256),
        # very large heads, spread over the chip
        _case("lstm_train_1x2048_b16_t256", "train", "lstm", "bf16", 256, 16, 1, 2048),
        # a wide layer in heads of 256, long context
        _case("slstm_train_8x256_b32_t2048", "train", "slstm", "bf16", 2048, 32, 8, 256, init=True),
        # one head, large batch: the top of the batch-size sweep
        _case("lstm_train_1x768_b128_t1024", "train", "lstm", "bf16", 1024, 128, 1, 768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: every cell, both data types, sequences of 1 to 2048 steps, batches of 1 to 256 rows, heads of 16 to
    2048 units (a multiple of 16; up to 256 with float32), at most as much work as the largest listed cases."""
    largest = [work(c) for c in listed()]
    max_bytes, max_flops = max(w["bytes"] for w in largest), max(w["flops"] for w in largest)
    while True:
        mode = rng.choices(["infer", "train", "recompute", "decode"], [3, 6, 2, 1])[0]
        cell = rng.choices(["lstm", "slstm", "gru", "elman", "gru4"], [5, 5, 3, 1, 1])[0]
        dtype = "bf16" if mode == "decode" or rng.random() < 0.8 else "f32"
        D = 16 * _log_int(rng, 1, 16 if dtype == "f32" else 128)
        NH = _log_int(rng, 1, 48)
        B = _log_int(rng, 1, 256)
        T = _log_int(rng, 1, 16) if mode == "decode" else _log_int(rng, 8, 2048)
        if mode == "decode" and (D > 1024 or NH * D * D > 1 << 20):   # the library's own scratch memory holds the packed weights of no more
            continue
        if NH * D > 2048 or T * D > 1024 * 768 or (T > 1024 and D > 256):
            continue
        case = _case("", mode, cell, dtype, T, B, NH, D, init=mode == "decode" or rng.random() < 0.5,
                     last=mode in ("train", "recompute") and rng.random() < 0.25,
                     clip=rng.choice([0.0, 0.0, 0.0, 1.0]) if mode in ("train", "recompute") else 0.0)
        del case["name"]
        # the serial chain, times the rounds over the batch that a large head needs, costs no more than the largest case's
        if T * D * math.ceil(B * NH * D / (128 * 768)) > 1024 * 768:
            continue
        w = work(case)
        if w["bytes"] <= max_bytes and w["flops"] <= max_flops:
            return case


def prepare(case, seed):
    T, B, NH, D = case["T"], case["B"], case["NH"], case["D"]
    cell, mode = case["cell"], case["mode"]
    G, S = GATES[cell], STATES[cell]
    io = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * scale).to(io)

    def uniform(lo, hi, *shape):
        return torch.rand(shape, generator=gen, device="cuda") * (hi - lo) + lo

    st = {"case": case, "cell": CELLS[cell]}
    st["Wx"] = normal(T, B, G, NH, D)
    st["R"] = normal(NH, D, G, D, scale=D ** -0.5)
    b = uniform(-0.1, 0.1, NH, G, D)
    if cell in ("lstm", "slstm"):   # forget biases spread over the heads
        b[:, FORGET, :] = torch.linspace(3.0, 6.0, NH, device="cuda")[:, None] if cell == "slstm" else 1.0
    st["b"] = b.to(io)
    st["states0"] = None
    if case["init"]:
        s0 = uniform(-0.5, 0.5, S, B, NH, D)
        if cell == "slstm":   # a cell in the middle of a sequence: |c| <= n, stabilizer at zero
            s0[2] += 1.0
            s0[1] *= s0[2]
            s0[3] = 0.0
        st["states0"] = s0
    desc = api.make_desc(CELLS[cell], 1 if mode == "decode" else T, B, NH, D, api.FLASHRNN_BF16 if case["dtype"] == "bf16" else api.FLASHRNN_F32)
    steps = 1 if mode == "decode" else T
    if mode == "decode":
        st["states"] = [torch.empty((2, S, B, NH, D), dtype=torch.float32, device="cuda") for _ in range(T)]
        return st
    st["states"] = torch.empty((steps + 1, S, B, NH, D), dtype=torch.float32, device="cuda")
    st["workspace"] = api.alloc_workspace(desc, "cuda")
    if mode == "infer":
        return st
    st["dH"] = normal(T, B, NH, D)
    st["dlast"] = uniform(-1.0, 1.0, S, B, NH, D) if case["last"] else None
    st["out"] = (torch.empty((T, B, G, NH, D), dtype=io, device="cuda"), torch.empty((NH, D, G, D), dtype=torch.float32, device="cuda"),
                 torch.empty((NH, G, D), dtype=torch.float32, device="cuda"), torch.empty((S, B, NH, D), dtype=torch.float32, device="cuda"))
    if mode == "train":
        st["cache"] = torch.empty(api.flashrnn_gate_cache_bytes(desc), dtype=torch.uint8, device="cuda")
    else:
        st["recompute_workspace"] = torch.zeros(api.lib().flashrnn_recompute_workspace_bytes(ctypes.byref(desc)), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    case, cell = st["case"], st["cell"]
    if case["mode"] == "decode":
        prev = st["states0"]
        for t, states in enumerate(st["states"]):
            api.flashrnn_fwd_static_scratch(cell, st["Wx"][t:t + 1], st["R"], st["b"], prev, save_for_backward=False, states=states)
            prev = states[1]
        return st["states"]
    train = case["mode"] == "train"
    states, cache, ws = api.flashrnn_fwd(cell, st["Wx"], st["R"], st["b"], st["states0"], save_for_backward=train, workspace=st["workspace"],
                                         states=st["states"], gate_cache=st.get("cache"))
    if case["mode"] == "infer":
        return states
    if train:
        grads = api.flashrnn_bwd(cell, st["R"], st["b"], states, cache, st["dH"], st["dlast"], workspace=ws, out=st["out"], recurrent_grad_clip=case["clip"])
    else:
        grads = api.flashrnn_bwd_recompute(cell, st["Wx"], st["R"], st["b"], states, st["dH"], st["dlast"], workspace=st["recompute_workspace"],
                                           out=st["out"], recurrent_grad_clip=case["clip"])[:4]
    return (states,) + tuple(grads)


def work(case):
    """Inputs once, outputs once; the recurrent product and, in training, its two transposes (once more where it is recomputed)."""
    T, B, H, D = case["T"], case["B"], case["NH"] * case["D"], case["D"]
    G, S, e = GATES[case["cell"]], STATES[case["cell"]], 2 if case["dtype"] == "bf16" else 4
    weights = H * G * D
    per_step = G * H * e + S * H * 4
    flops = 2 * T * B * weights
    if case["mode"] == "decode":   # every call reads the weights anew
        return {"bytes": T * (B * per_step + weights * e), "flops": flops}
    if case["mode"] == "infer":
        return {"bytes": T * B * per_step + weights * e, "flops": flops}
    per_step += H * e + G * H * e
    return {"bytes": T * B * per_step + weights * (e + 4), "flops": flops * (4 if case["mode"] == "recompute" else 3)}


def tolerance(case):
    """About four times the largest relative error of any output against the same path in 64 bits: with bf16 inputs and outputs, whose
    rounding of the products' operands dominates, 1e-3 on states and 2e-3 to 4.3e-3 on gradients (sequences of 9 to 1628 steps); with
    float32, 1e-7 on states and up to 6e-7 on weight gradients, which sum tens of thousands of terms."""
    return {"rel": 1.5e-2 if case["dtype"] == "bf16" else 5e-6}
