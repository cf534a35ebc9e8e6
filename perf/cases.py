"""The work that programs using the compensated quantized linear have it do.

Six kinds of pass, each through the public entry points of
``paper_2605_05819_amd.cl``:

``linear``    one compensated linear on a few decode tokens, called eagerly.
``layer``     decoder layers (Q/K/V window, O, gated gate/up window, down) on a
              few decode tokens.  A serving program captures its decode step
              once as a HIP graph and replays it for every token, so the state
              holds the captured step and a pass replays it.
``prefill``   one compensated linear on a prompt's tokens, called eagerly.
``moe``       mixture-of-experts layers (gate/up window, gated down) on a few
              decode tokens, captured and replayed as ``layer`` is.
``quantize``  a weight to its packed backbone, and the backbone back to float32.
``factors``   the compensation factors and spectrum of a quantized weight.

Weights are N(0, 0.02^2) rounded to nearest on the per-group min/max grid,
activations N(0, 1), routing the top k of a softmax over N(0, 1) logits.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2605_05819_amd import cl

DEV = "cuda"
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}
# Ranks of q, k, v, o, gate, up, down: one allocator result for each code width.
RANKS = {4: "32,64,64,32,64,128,32", 3: "128,64,0,0,128,64,32", 2: "64,128,64,64,64,256,128"}


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest call: one 1024 x 1024 linear, one token, rank 16.
        {"name": "linear-1024-T1", "kind": "linear", "d_out": 1024, "d_in": 1024, "bits": 4, "group": 128,
         "r_max": 16, "rank": 16, "T": 1, "act": "fp16", "out": "fp16"},
        # Single-stream decoding of a Llama-3.1-8B-shaped model at 4 bits.
        {"name": "layer-w4-T1", "kind": "layer", "layers": 4, "hidden": 4096, "kv": 1024, "ffn": 14336, "bits": 4,
         "group": 128, "r_max": 128, "ranks": RANKS[4], "T": 1, "act": "fp16"},
        # The aggressive 2-bit backbone with groups of 64 and ranks up to 256.
        {"name": "layer-w2-T1", "kind": "layer", "layers": 4, "hidden": 4096, "kv": 1024, "ffn": 14336, "bits": 2,
         "group": 64, "r_max": 256, "ranks": RANKS[2], "T": 1, "act": "fp16"},
        # A small serving batch on the INT3 backbone, bf16 activations.
        {"name": "layer-w3-T4", "kind": "layer", "layers": 4, "hidden": 4096, "kv": 1024, "ffn": 14336, "bits": 3,
         "group": 128, "r_max": 128, "ranks": RANKS[3], "T": 4, "act": "bf16"},
        # An ordinary serving batch at 4 bits.
        {"name": "layer-w4-T16", "kind": "layer", "layers": 4, "hidden": 4096, "kv": 1024, "ffn": 14336, "bits": 4,
         "group": 128, "r_max": 128, "ranks": RANKS[4], "T": 16, "act": "fp16"},
        # A 2048-token prompt through the widest projection: the largest product.
        {"name": "prefill-gate-M2048", "kind": "prefill", "d_out": 14336, "d_in": 4096, "bits": 4, "group": 128,
         "r_max": 128, "rank": 64, "M": 2048, "act": "bf16", "out": "bf16"},
        # A short prompt of odd length through a square INT3 projection.
        {"name": "prefill-o-M333", "kind": "prefill", "d_out": 4096, "d_in": 4096, "bits": 3, "group": 128,
         "r_max": 128, "rank": 32, "M": 333, "act": "fp16", "out": "fp16"},
        # Single-stream decoding of Qwen3-30B-A3B-shaped experts.
        {"name": "moe-T1", "kind": "moe", "layers": 8, "E": 128, "k": 8, "hidden": 2048, "ffn": 768, "bits": 4,
         "group": 128, "r_max": 32, "T": 1, "slot_ranks": False, "act": "fp16"},
        # A small batch, ranks per slot (the expert-activation term).
        {"name": "moe-T8", "kind": "moe", "layers": 4, "E": 128, "k": 8, "hidden": 2048, "ffn": 768, "bits": 4,
         "group": 128, "r_max": 32, "T": 8, "slot_ranks": True, "act": "bf16"},
        # The largest decode batch: most experts are routed, several slots each.
        {"name": "moe-T64", "kind": "moe", "layers": 4, "E": 128, "k": 8, "hidden": 2048, "ffn": 768, "bits": 4,
         "group": 128, "r_max": 32, "T": 64, "slot_ranks": False, "act": "fp16"},
        # Preparing a model: its widest projection to 4 bits and back (what the
        # residual and every check of a quantized model read).
        {"name": "quantize-gate", "kind": "quantize", "d_out": 14336, "d_in": 4096, "bits": 4, "group": 128},
        # Preparing a model: the factors of a k or v projection.  The square
        # projections take the same path for seconds each.
        {"name": "factors-kv", "kind": "factors", "d_out": 1024, "d_in": 4096, "bits": 3, "group": 128,
         "r_max": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _group(rng, bits):
    return rng.choice({4: (32, 64, 128), 3: (32, 64, 128), 2: (64, 128)}[bits])


def draw(rng):
    kind = rng.choice(("linear", "layer", "layer", "prefill", "prefill", "moe", "moe", "quantize", "factors"))
    bits = rng.choice((4, 4, 3, 2))
    group = _group(rng, bits)
    act = rng.choice(("fp16", "bf16"))
    if kind == "linear":
        r_max = rng.choice((16, 32, 64, 128, 256))
        return {"kind": kind, "d_out": _log(rng, 64, 16384), "d_in": 128 * _log(rng, 2, 112), "bits": bits,
                "group": group, "r_max": r_max, "rank": rng.randint(0, r_max), "T": _log(rng, 1, 64), "act": act,
                "out": rng.choice(("fp16", "bf16", "fp32"))}
    if kind == "layer":
        hidden = 256 * rng.randint(4, 16)
        r_max = rng.choice((64, 128))
        return {"kind": kind, "layers": rng.randint(1, 4), "hidden": hidden, "kv": rng.choice((256, 512, 1024)),
                "ffn": 128 * rng.randint(hidden // 64, 7 * hidden // 256), "bits": bits, "group": group,
                "r_max": r_max, "ranks": ",".join(str(rng.choice((0, 16, 32, 64, r_max))) for _ in range(7)),
                "T": _log(rng, 1, 64), "act": act}
    if kind == "prefill":
        d_out, d_in = _log(rng, 256, 14336), 128 * _log(rng, 4, 112)
        M = min(_log(rng, 16, 4096), 2048 * 14336 * 4096 // (d_out * d_in))
        r_max = rng.choice((32, 64, 128))
        return {"kind": kind, "d_out": d_out, "d_in": d_in, "bits": bits, "group": group, "r_max": r_max,
                "rank": rng.randint(0, r_max), "M": M, "act": act, "out": rng.choice((act, "fp32"))}
    if kind == "moe":
        bits = rng.choice((4, 4, 2))
        group = rng.choice((64, 128))
        E = _log(rng, 8, 160)
        return {"kind": kind, "layers": rng.randint(1, 4), "E": E, "k": rng.randint(1, 8),
                "hidden": 128 * rng.randint(4, 16), "ffn": 128 * rng.randint(2, 6), "bits": bits, "group": group,
                "r_max": rng.choice((16, 32, 64)), "T": _log(rng, 1, 64), "slot_ranks": rng.random() < 0.5, "act": act}
    if kind == "quantize":
        return {"kind": kind, "d_out": _log(rng, 64, 14336), "d_in": 128 * _log(rng, 2, 32), "bits": bits,
                "group": group}
    small, large = _log(rng, 48, 1024), 128 * _log(rng, 8, 32)
    if rng.random() < 0.3:
        return {"kind": kind, "d_out": large + rng.randint(0, 63) if large < 4096 else large,
                "d_in": 128 * max(1, small // 128), "bits": bits, "group": group, "r_max": rng.randint(1, min(small // 2, 128))}
    return {"kind": kind, "d_out": small, "d_in": large, "bits": bits, "group": group,
            "r_max": rng.randint(1, min(small, 128))}


# ------------------------------------------------------------------ the inputs

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(gen, shape, std, dtype):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).mul_(std).to(dtype)


def _pack(codes, bits):
    """int32 codes [..][n] -> the bit string in 32-bit words [..][n bits / 32]."""
    if bits == 3:
        c = codes.view(*codes.shape[:-1], -1, 32).to(torch.int64)
        words = torch.zeros(*c.shape[:-1], 3, dtype=torch.int64, device=c.device)
        for i in range(32):
            w, off = (3 * i) // 32, (3 * i) % 32
            words[..., w] |= (c[..., i] << off) & 0xFFFFFFFF
            if off > 29:
                words[..., w + 1] |= c[..., i] >> (32 - off)
        words = torch.where(words >= 1 << 31, words - (1 << 32), words)
        return words.to(torch.int32).flatten(-2).contiguous()
    per = 32 // bits
    c = codes.view(*codes.shape[:-1], -1, per)
    words = torch.zeros(c.shape[:-1], dtype=torch.int32, device=c.device)
    for i in range(per):
        words |= c[..., i] << (bits * i)
    return words.contiguous()


def _backbone(gen, lead, d_in, bits, group):
    """A weight [*lead][d_in] rounded to nearest on its per-group grid: the
    packed words, the fp16 scales and zeros, and (codes - zero) scale as a
    function, for the 64-bit values."""
    w = _normal(gen, (*lead, d_in // group, group), 0.02, torch.float32)
    qmax = (1 << bits) - 1
    lo, hi = w.amin(-1).clamp_(max=0), w.amax(-1).clamp_(min=0)
    s = ((hi - lo) / qmax).to(torch.float16)
    sf = s.float()
    z = (-lo / sf).round_().clamp_(0, qmax)
    codes = (w.div_(sf[..., None]).round_() + z[..., None]).clamp_(0, qmax).to(torch.int32)
    q = _pack(codes.view(*lead, d_in), bits)

    def exact(index=None):
        c, zz, ss = (codes, z, sf) if index is None else (codes[index], z[index], sf[index])
        return ((c.double() - zz.double()[..., None]) * ss.double()[..., None]).flatten(-2)

    return q, s, z.to(torch.float16), exact


def _factors(gen, lead, d_out, d_in, r_max):
    return (_normal(gen, (*lead, r_max, d_in), 0.01, torch.float16),
            _normal(gen, (*lead, d_out, r_max), 0.01, torch.float16))


def _linear(gen, d_out, d_in, case, rank):
    q, s, z, exact = _backbone(gen, (d_out,), d_in, case["bits"], case["group"])
    A, B = _factors(gen, (), d_out, d_in, case["r_max"])
    w = cl.QWeight(q, s, z, d_out, d_in, case["bits"], case["group"])
    return SimpleNamespace(w=w, c=cl.LowRank(A, B, case["r_max"], rank), exact=exact)


def _linear_exact(lin, x):
    y = x @ lin.exact().T
    r = lin.c.rank
    if r:
        y += (x @ lin.c.A[:r].double().T) @ lin.c.B[:, :r].double().T
    return y


def _layer_shapes(case):
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return ((h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f))


def _layer_inputs(case, seed):
    """Layers of linears q, k, v, o, gate, up, down, with the inputs of the
    attention, of o and of the MLP."""
    gen, ranks = _generator(seed), [int(r) for r in case["ranks"].split(",")]
    for _ in range(case["layers"]):
        mats = [_linear(gen, d_out, d_in, case, r) for (d_out, d_in), r in zip(_layer_shapes(case), ranks)]
        xs = [_normal(gen, (case["T"], case["hidden"]), 1.0, DTYPES[case["act"]]) for _ in range(3)]
        yield mats, xs


def _moe_inputs(case, seed):
    """Layers of stacked experts gate, up, down, with the layer's input, the
    routing and (for slot_ranks) the ranks of the slots."""
    gen = _generator(seed)
    E, k, T, h, f, r_max = (case[n] for n in ("E", "k", "T", "hidden", "ffn", "r_max"))
    levels = torch.tensor([0, r_max // 4, r_max // 2, r_max], dtype=torch.int32, device=DEV)
    for _ in range(case["layers"]):
        mats = []
        for d_out, d_in in ((f, h), (f, h), (h, f)):
            q, s, z, exact = _backbone(gen, (E, d_out), d_in, case["bits"], case["group"])
            A, B = _factors(gen, (E,), d_out, d_in, r_max)
            ranks = levels[torch.randint(0, 4, (E,), generator=gen, device=DEV)]
            mats.append(SimpleNamespace(ex=cl.MoeExperts(q, s, z, A, B, ranks, E, d_out, d_in, case["bits"],
                                                         case["group"], r_max), exact=exact))
        x = _normal(gen, (T, h), 1.0, DTYPES[case["act"]])
        p, ids = torch.softmax(_normal(gen, (T, E), 1.0, torch.float32), -1).topk(min(k, E), -1)
        slots = [None] * 3
        if case["slot_ranks"]:
            share = k * p / p.sum(-1, keepdim=True)
            slots = [(share * m.ex.ranks[ids]).round().clamp(max=r_max).to(torch.int32).contiguous() for m in mats]
        yield mats, x, ids.to(torch.int32).contiguous(), slots


def _captured(state, step):
    """The step as a HIP graph, as a serving program captures it."""
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        step()
    torch.cuda.synchronize()
    state.graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(state.graph, stream=stream):
        step()
    torch.cuda.synchronize()
    return state


def _prepare_layer(case, seed):
    act, T, f = DTYPES[case["act"]], case["T"], case["ffn"]
    state = SimpleNamespace(kind="layer", outputs=[])
    calls = []
    for mats, xs in _layer_inputs(case, seed):
        windows = [[m.w for m in g] for g in (mats[0:3], mats[3:4], mats[4:6], mats[6:7])]
        factors = [[m.c for m in g] for g in (mats[0:3], mats[3:4], mats[4:6], mats[6:7])]
        wss = [cl.workspace(cl.window_workspace(w, c, T), DEV) for w, c in zip(windows, factors)]
        ys = [torch.empty((T, m.w.d_out), dtype=act, device=DEV) for m in mats[0:4] + mats[6:7]]
        h = torch.empty((T, f), dtype=act, device=DEV)
        calls.append((windows, factors, wss, xs, ys, h))
        state.outputs.append(ys + [h])

    def step():
        for windows, factors, wss, xs, ys, h in calls:
            cl.linear_decode_window(windows[0], factors[0], xs[0], ys=ys[0:3], ws=wss[0])
            cl.linear_decode(windows[1][0], factors[1][0], xs[1], y=ys[3], ws=wss[1])
            cl.linear_decode_glu(windows[2], factors[2], xs[2], h=h, ws=wss[2])
            cl.linear_decode(windows[3][0], factors[3][0], h, y=ys[4], ws=wss[3])

    state.calls = calls
    return _captured(state, step)


def _prepare_moe(case, seed):
    act, T = DTYPES[case["act"]], case["T"]
    state = SimpleNamespace(kind="moe", outputs=[])
    calls = []
    for mats, x, ids, slots in _moe_inputs(case, seed):
        gate, up, down = (m.ex for m in mats)
        k = ids.shape[1]
        gu = [torch.empty((T, k, case["ffn"]), dtype=act, device=DEV) for _ in range(2)]
        y = torch.empty((T, k, case["hidden"]), dtype=act, device=DEV)
        ws = (cl.workspace(cl.moe_window_workspace([gate, up], T, k, False), DEV),
              cl.workspace(cl.moe_gated_workspace(down, T, k), DEV))
        calls.append((gate, up, down, x, ids, slots, gu, y, ws))
        state.outputs.append(gu + [y])

    def step():
        for gate, up, down, x, ids, slots, gu, y, ws in calls:
            cl.moe_linear_decode_window([gate, up], x, ids, ys=gu, ws=ws[0],
                                        slot_ranks=None if slots[0] is None else slots[:2])
            cl.moe_linear_decode_gated(down, gu[0], gu[1], ids, y=y, ws=ws[1], slot_ranks=slots[2])

    state.calls = calls
    return _captured(state, step)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "layer":
        return _prepare_layer(case, seed)
    if kind == "moe":
        return _prepare_moe(case, seed)
    gen = _generator(seed)
    d_out, d_in, bits, group = (case[n] for n in ("d_out", "d_in", "bits", "group"))
    if kind in ("quantize", "factors"):
        W = _normal(gen, (d_out, d_in), 0.02, torch.float32)
        state = SimpleNamespace(kind=kind, W=W, bits=bits, group=group)
        if kind == "factors":
            state.w, state.r_max = cl.quantize_pack(W, bits, group), case["r_max"]
        return state
    tokens = case["T"] if kind == "linear" else case["M"]
    lin = _linear(gen, d_out, d_in, case, case["rank"])
    need = cl.linear_workspace if kind == "linear" else cl.prefill_workspace
    return SimpleNamespace(kind=kind, w=lin.w, c=lin.c, x=_normal(gen, (tokens, d_in), 1.0, DTYPES[case["act"]]),
                           y=torch.empty((tokens, d_out), dtype=DTYPES[case["out"]], device=DEV),
                           ws=cl.workspace(need(lin.w, lin.c, tokens), DEV))


# -------------------------------------------------------------------- the pass

def run(state):
    if state.kind in ("layer", "moe"):
        state.graph.replay()
        return state.outputs
    if state.kind == "linear":
        return cl.linear_decode(state.w, state.c, state.x, y=state.y, ws=state.ws)
    if state.kind == "prefill":
        return cl.linear_prefill(state.w, state.c, state.x, Y=state.y, ws=state.ws)
    if state.kind == "quantize":
        w = cl.quantize_pack(state.W, state.bits, state.group)
        return w.q, w.scales, w.zeros, cl.dequantize(w)
    return cl.build_compensation(state.W, state.w, state.r_max)


# ------------------------------------------------------- what a pass needs to do

def _linear_bytes(d_out, d_in, case, rank, tokens, out=2):
    return (d_out * d_in * case["bits"] // 8 + 4 * d_out * d_in // case["group"] + 2 * rank * (d_in + d_out) +
            tokens * (2 * d_in + out * d_out))


def _linear_flops(d_out, d_in, rank, tokens):
    return 2 * tokens * (d_out * d_in + rank * (d_in + d_out))


def work(case):
    kind = case["kind"]
    if kind == "layer":
        T, ranks = case["T"], [int(r) for r in case["ranks"].split(",")]
        shapes = list(zip(_layer_shapes(case), ranks))
        # q, k and v read one input, and so do gate and up, which write one output
        shared = 2 * T * (3 * case["hidden"] + case["ffn"])
        return {"bytes": case["layers"] * (sum(_linear_bytes(o, i, case, r, T) for (o, i), r in shapes) - shared),
                "flops": case["layers"] * sum(_linear_flops(o, i, r, T) for (o, i), r in shapes)}
    if kind == "moe":
        E, k, T, h, f = (case[n] for n in ("E", "k", "T", "hidden", "ffn"))
        k = min(k, E)
        routed = E * (1 - (1 - k / E) ** T)
        rank = 7 * case["r_max"] // 16
        per = sum(_linear_bytes(o, i, case, rank, 0) for o, i in ((f, h), (f, h), (h, f)))
        return {"bytes": case["layers"] * (routed * per + T * (2 * h + k * (4 * f + 4 * f + 2 * h))),
                "flops": case["layers"] * sum(_linear_flops(o, i, rank, T * k) for o, i in ((f, h), (f, h), (h, f)))}
    d_out, d_in = case["d_out"], case["d_in"]
    if kind == "quantize":
        packed = d_out * d_in * case["bits"] // 8 + 4 * d_out * d_in // case["group"]
        return {"bytes": 8 * d_out * d_in + 2 * packed, "flops": 6 * d_out * d_in}
    if kind == "factors":
        # the Gram matrix, the eigenvalues by a reduction to tridiagonal form,
        # the leading vectors back through it and through the residual
        n, r = min(d_out, d_in), case["r_max"]
        return {"bytes": 4 * d_out * d_in + d_out * d_in * case["bits"] // 8 + 4 * d_out * d_in // case["group"] +
                2 * r * (d_out + d_in) + 4 * n,
                "flops": d_out * d_in * n + 4 * n ** 3 // 3 + 2 * r * n * n + 2 * r * d_out * d_in}
    tokens = case["T"] if kind == "linear" else case["M"]
    return {"bytes": _linear_bytes(d_out, d_in, case, case["rank"], tokens, 4 if case["out"] == "fp32" else 2),
            "flops": _linear_flops(d_out, d_in, case["rank"], tokens)}


# ---------------------------------------------------------------- right results

def tolerance(case):
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "factors":
        return {"rel": 1e-3}
    if kind == "prefill":
        # the weight tile is rounded to fp16 once, then the result to its type
        return {"rel": {"fp32": 8e-4, "fp16": 1e-3, "bf16": 7e-3}[case["out"]]}
    if kind == "linear":
        return {"rel": {"fp32": 1.2e-5, "fp16": 9e-4, "bf16": 7e-3}[case["out"]]}
    # the MLP's input to its down projection, and the experts' gate and up
    # outputs, are rounded on the way
    return {"rel": {"layer": {"fp16": 1.2e-3, "bf16": 1e-2}, "moe": {"fp16": 1.8e-3, "bf16": 1.2e-2}}[kind][case["act"]]}


def _layer_exact(case, seed):
    layers = []
    for mats, xs in _layer_inputs(case, seed):
        xs = [x.double() for x in xs]
        ys = [_linear_exact(m, xs[0]) for m in mats[0:3]] + [_linear_exact(mats[3], xs[1])]
        h = torch.nn.functional.silu(_linear_exact(mats[4], xs[2])) * _linear_exact(mats[5], xs[2])
        layers.append(ys + [_linear_exact(mats[6], h), h])
    return layers


def _moe_exact(case, seed):
    def apply(m, x, ids, ranks):
        """x [T][k][d_in] in 64 bits -> [T][k][d_out], one expert at a time."""
        y = torch.zeros((*ids.shape, m.ex.d_out), dtype=torch.float64, device=DEV)
        column = torch.arange(m.ex.r_max, device=DEV)
        for e in ids.unique().tolist():
            at = ids == e
            t = x[at] @ m.ex.A[e].double().T
            t = torch.where(column < ranks[at][:, None], t, torch.zeros_like(t))
            y[at] = x[at] @ m.exact(e).T + t @ m.ex.B[e].double().T
        return y

    layers = []
    for mats, x, ids, slots in _moe_inputs(case, seed):
        ids = ids.long()
        ranks = [m.ex.ranks[ids] if s is None else s for m, s in zip(mats, slots)]
        xk = x.double()[:, None].expand(-1, ids.shape[1], -1)
        g, u = (apply(m, xk, ids, r) for m, r in zip(mats[:2], ranks))
        y = apply(mats[2], torch.nn.functional.silu(g) * u, ids, ranks[2])
        layers.append([g, u, y])
    return layers


def _grid(W, bits, group):
    """The per-group grid in 64 bits, the step rounded once to fp16."""
    d_out, d_in = W.shape
    qmax = (1 << bits) - 1
    w = W.double().view(d_out, d_in // group, group)
    lo, hi = w.amin(-1).clamp_(max=0), w.amax(-1).clamp_(min=0)
    s = torch.from_numpy(((hi - lo) / qmax).cpu().numpy().astype(np.float16).astype(np.float64)).to(DEV)
    z = (-lo / s).round().clamp_(0, qmax)
    hat = (((w / s[..., None]).round() + z[..., None]).clamp_(0, qmax) - z[..., None]) * s[..., None]
    return s, z, hat.view(d_out, d_in)


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        return _layer_exact(case, seed)
    if kind == "moe":
        return _moe_exact(case, seed)
    gen = _generator(seed)
    d_out, d_in = case["d_out"], case["d_in"]
    if kind in ("quantize", "factors"):
        W = _normal(gen, (d_out, d_in), 0.02, torch.float32)
        s, z, hat = _grid(W, case["bits"], case["group"])
        if kind == "quantize":
            return None, s, z, hat
        U, sigma, Vt = (torch.from_numpy(v) for v in
                        np.linalg.svd((W.double() - hat).cpu().numpy(), full_matrices=False))
        r = case["r_max"]
        U, Vt, root = U[:, :r], Vt[:r], sigma[:r].sqrt()
        sign = torch.sign(U.gather(0, U.abs().argmax(0, keepdim=True)))
        return (sign * root).T * Vt, U * (sign * root), sigma
    lin = _linear(gen, d_out, d_in, case, case["rank"])
    x = _normal(gen, (case["T"] if kind == "linear" else case["M"], d_in), 1.0, DTYPES[case["act"]])
    return _linear_exact(lin, x.double())
