"""The work this library is timed on, through its public entry points.

Every case is something a serving program does with the nested layers: a
decode pass over a transformer layer set replayed from its captured graph, a
prefill pass, a grouped (MoE) layer, one small layer called eagerly, and the
loading of a layer (encoding choice and split).  listed() names twelve of
them, draw() gives more of the same ranges, odd sizes among them.

Inputs are drawn on the GPU from the seed alone: weights N(0, 0.02^2) as FP16,
activations N(0, 1) as FP16 (prefill: 1% of the channels times 20), residual
chunks in place or at random slots of a pool twice the size.
"""
import math

import torch

from paper_2609_34380_amd import dps, graphs

# (N = output features, K = input features) of QKV, O, gate+up and down
SETS = {
    "h4096": ((6144, 4096), (4096, 4096), (28672, 4096), (4096, 14336)),
    "h8192": ((10240, 8192), (8192, 8192), (57344, 8192), (8192, 28672)),
}
MODES = {"full": dps.MODE_FULL, "fast": dps.MODE_FAST}
ENCS = {"e5m2": dps.ENC_E5M2, "e4m3": dps.ENC_E4M3}


def listed():
    return [
        # one small layer, a handful of tokens, called eagerly: launch and host latency
        {"name": "layer_1024_m4_full", "kind": "layer", "n": 1024, "k": 1024, "m": 4,
         "mode": "full", "enc": "e5m2", "act": "fp16", "log2_chunk": 16, "scattered": False},
        # one user, one token a step: the weight stream alone
        {"name": "decode_m1_full", "kind": "decode", "set": "h4096", "m": 1, "mode": "full",
         "enc": "e5m2", "log2_chunk": 21, "scattered": False},
        # a small batch while KV blocks hold the residual region
        {"name": "decode_m8_fast", "kind": "decode", "set": "h4096", "m": 8, "mode": "fast",
         "enc": "e5m2", "log2_chunk": 21, "scattered": False},
        # an ordinary decode batch at full precision, layers nested as E4M3
        {"name": "decode_m32_full_e4m3", "kind": "decode", "set": "h4096", "m": 32,
         "mode": "full", "enc": "e4m3", "log2_chunk": 21, "scattered": False},
        # a larger model whose residual chunks sit between KV blocks
        {"name": "decode_h8192_m64_full", "kind": "decode", "set": "h8192", "m": 64,
         "mode": "full", "enc": "e5m2", "log2_chunk": 21, "scattered": True},
        # a burst served in fast mode
        {"name": "decode_m128_fast", "kind": "decode", "set": "h4096", "m": 128, "mode": "fast",
         "enc": "e5m2", "log2_chunk": 21, "scattered": False},
        # the largest captured decode batch, full precision
        {"name": "decode_m256_full", "kind": "decode", "set": "h4096", "m": 256, "mode": "full",
         "enc": "e5m2", "log2_chunk": 21, "scattered": False},
        # a prompt of ordinary, ragged length at full precision
        {"name": "prefill_1531_full", "kind": "prefill", "set": "h4096", "m": 1531,
         "mode": "full", "enc": "e5m2", "act": "fp16", "log2_chunk": 21, "scattered": False},
        # a long prompt (or several) in fast mode on FP8 activations: the largest call
        {"name": "prefill_8192_fp8", "kind": "prefill", "set": "h4096", "m": 8192,
         "mode": "fast", "enc": "e5m2", "act": "fp8", "log2_chunk": 21, "scattered": False},
        # a mixed batch through a layer of 8 experts, two of them per token
        {"name": "moe_512_full", "kind": "moe", "experts": 8, "hidden": 4096, "ffn": 14336,
         "tokens": 512, "topk": 2, "mode": "full", "enc": "e5m2", "act": "fp16",
         "log2_chunk": 21, "scattered": False},
        # a decode batch through the same layer: a few rows per expert
        {"name": "moe_16_fast", "kind": "moe", "experts": 8, "hidden": 4096, "ffn": 14336,
         "tokens": 16, "topk": 2, "mode": "fast", "enc": "e5m2", "act": "fp16",
         "log2_chunk": 21, "scattered": False},
        # loading a layer: the encoding its weights admit, then the two planes
        {"name": "load_gate_up", "kind": "load", "n": 28672, "k": 4096, "enc": "e4m3",
         "log2_chunk": 21, "scattered": True},
    ]


def _log(rng, lo, hi):
    """A whole number in lo .. hi, spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    case = {"kind": rng.choice(("layer", "decode", "decode", "prefill", "moe", "load", "unload")),
            "enc": rng.choice(("e5m2", "e5m2", "e4m3")), "log2_chunk": rng.choice((14, 16, 21, 21)),
            "scattered": rng.random() < 0.5}
    kind = case["kind"]
    if kind == "layer":
        case.update(n=_log(rng, 200, 30000), k=16 * _log(rng, 16, 900), m=_log(rng, 1, 600))
    elif kind == "decode":
        case.update(set=rng.choice(("h4096", "h4096", "h8192")), m=_log(rng, 1, 256))
    elif kind == "prefill":
        case.update(set="h4096", m=_log(rng, 257, 4096))
    elif kind == "moe":
        hidden, ffn, experts = rng.choice(((4096, 14336, 8), (2048, 1536, 32), (3072, 4112, 16)))
        case.update(hidden=hidden, ffn=ffn, experts=experts, topk=2, tokens=_log(rng, 4, 1500))
    else:
        case.update(n=_log(rng, 500, 30000), k=16 * _log(rng, 32, 900))
        return case
    case["mode"] = rng.choice(("full", "fast"))
    if kind != "decode":
        case["act"] = "fp16" if case["mode"] == "full" else rng.choice(("fp16", "fp8"))
    return case


# ---- inputs ---------------------------------------------------------------------


def _shapes(case):
    if "set" in case:
        return SETS[case["set"]]
    if case["kind"] == "moe":
        return ((2 * case["ffn"], case["hidden"]), (case["hidden"], case["ffn"]))
    return ((case["n"], case["k"]),)


def _rows(case):
    return case["tokens"] * case["topk"] if case["kind"] == "moe" else case["m"]


def _gen(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * int(seed) + part)
    return g


def _weights(case, seed, layer):
    n, k = _shapes(case)[layer]
    shape = (case["experts"], n, k) if case["kind"] == "moe" else (n, k)
    w = torch.empty(shape, dtype=torch.float16, device="cuda")
    return w.normal_(0.0, 0.02, generator=_gen(seed, 10 + layer))


def _activations(case, seed, layer):
    m, k = _rows(case), _shapes(case)[layer][1]
    g = _gen(seed, 50 + layer)
    x = torch.randn((m, k), generator=g, device="cuda")
    if case["kind"] == "prefill":  # outlier channels
        x[:, torch.randperm(k, generator=g, device="cuda")[: max(1, k // 100)]] *= 20.0
    return x.to(torch.float16)


def _offsets(case, seed):
    """Row offsets of each expert: every token goes to topk different experts."""
    g = _gen(seed, 90)
    score = torch.rand((case["tokens"], case["experts"]), generator=g, device="cuda")
    chosen = score.topk(case["topk"], dim=1).indices.reshape(-1)
    counts = torch.bincount(chosen, minlength=case["experts"])
    offsets = torch.zeros(case["experts"] + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = torch.cumsum(counts, 0)
    return offsets


def _residual(case, seed, numel, layer):
    chunks = -(-numel // (1 << case["log2_chunk"]))
    if case["scattered"]:
        slots = torch.randperm(2 * chunks, generator=_gen(seed, 30 + layer), device="cuda")[:chunks]
        slots = slots.to(torch.int32)
        pool = torch.zeros(2 * chunks << case["log2_chunk"], dtype=torch.uint8, device="cuda")
        return dps.make_residual(numel, case["log2_chunk"], "cuda", slots=slots, pool=pool)
    return dps.make_residual(numel, case["log2_chunk"], "cuda")


# ---- what a program has in hand, and one pass -------------------------------------

_stream = None


def _compute_stream():
    """The one stream a serving process replays its graphs on."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def prepare(case, seed):
    mode = MODES.get(case.get("mode"))
    enc = ENCS[case["enc"]]
    state = {"case": case, "mode": mode}
    if case["kind"] in ("load", "unload"):
        w = _weights(case, seed, 0)
        res = _residual(case, seed, w.numel(), 0)
        if case["kind"] == "load":
            state.update(w=w, res=res, enc=enc,
                         hi=torch.empty(w.shape, dtype=torch.uint8, device="cuda"))
        else:
            state.update(nw=dps.split(w, res, enc=enc), out=torch.empty_like(w))
        return state

    shapes, rows = _shapes(case), _rows(case)
    act = case.get("act", "fp16")
    state["nws"] = []
    for layer in range(len(shapes)):
        w = _weights(case, seed, layer)
        state["nws"].append(dps.split(w, _residual(case, seed, w.numel(), layer), enc=enc))
        del w
    state["xs"] = [_activations(case, seed, layer) for layer in range(len(shapes))]
    state["act"] = act
    if case["kind"] == "layer":
        return state  # called plainly: the binding makes output and workspace
    state["ys"] = [torch.zeros((rows, n), dtype=torch.float16, device="cuda") for n, _ in shapes]
    flag = dps.ACT_FP8_ROWSCALE if act == "fp8" else dps.ACT_FP16
    modes = (dps.MODE_FULL, dps.MODE_FAST) if case["kind"] == "decode" else (mode,)
    need = max(dps.workspace_bytes(md, flag, rows, n, k, case.get("experts", 1))
               for md in modes for n, k in shapes)
    state["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    if case["kind"] == "moe":
        state["offsets"] = _offsets(case, seed)
    if case["kind"] == "decode":
        def step(m, md, nws=state["nws"], xs=state["xs"], ys=state["ys"], ws=state["ws"]):
            for x, nw, y in zip(xs, nws, ys):
                dps.linear(x, nw, md, out=y, workspace=ws)
        state["graphs"] = graphs.ModeGraphs(step, (rows,), stream=_compute_stream()).capture()
    return state


def run(state):
    case, mode = state["case"], state["mode"]
    kind = case["kind"]
    if kind == "load":
        enc = dps.select_enc(state["w"])
        nw = dps.split(state["w"], state["res"], hi=state["hi"], enc=state["enc"])
        return [enc, nw.hi, state["res"].pool]
    if kind == "unload":
        return dps.merge(state["nw"], out=state["out"])
    if kind == "layer":
        return dps.linear(state["xs"][0], state["nws"][0], mode, act=state["act"])
    if kind == "decode":
        state["graphs"].replay(case["m"], mode)
    elif kind == "prefill":
        for x, nw, y in zip(state["xs"], state["nws"], state["ys"]):
            dps.linear(x, nw, mode, act=state["act"], out=y, workspace=state["ws"])
    else:
        for x, nw, y in zip(state["xs"], state["nws"], state["ys"]):
            dps.linear_grouped(x, state["offsets"], nw, mode, act=state["act"], out=y,
                               workspace=state["ws"])
    return state["ys"]


# ---- what a pass cannot do without, and what it has to give -------------------------


def work(case):
    shapes = _shapes(case)
    if case["kind"] in ("load", "unload"):
        n, k = shapes[0]
        return {"bytes": 4 * n * k, "flops": 0}
    rows = _rows(case)
    planes = 2 if case["mode"] == "full" else 1
    bytes_ = flops = 0
    for n, k in shapes:
        # an expert without rows reads nothing; fewer rows than experts leave some out
        experts = min(case["experts"], rows) if case["kind"] == "moe" else 1
        bytes_ += planes * experts * n * k + 2 * rows * (n + k)
        flops += 2 * rows * n * k
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] in ("load", "unload"):
        return "exact"
    # outputs are FP16: rounding alone is 2.1e-4 of their norm
    return {"rel": 8e-4, "max": 4e-3}


def _weights64(case, w):
    """The weights a mode multiplies by, in 64 bits: full mode the FP16 words;
    fast mode the words cut to two (E5M2) or three (E4M3) mantissa bits."""
    if case["mode"] == "fast":
        keep = -256 if case["enc"] == "e5m2" else -128  # 0xFF00, 0xFF80
        w = (w.view(torch.int16) & keep).view(torch.float16)
    return w.double()


def _activations64(case, x):
    """FP16 activations, or (FP8) E4M3 values times a power-of-two row scale."""
    if case.get("act", "fp16") != "fp8":
        return x.double()
    x = x.double()
    amax = x.abs().amax(dim=1, keepdim=True)
    scale = torch.where(amax > 0, torch.exp2(torch.ceil(torch.log2(amax / 448.0))), 1.0)
    return (x / scale).to(torch.float32).to(torch.float8_e4m3fn).double() * scale


def exact(case, seed):
    if case["kind"] == "load":
        return None
    if case["kind"] == "unload":
        return _weights(case, seed, 0)
    out = []
    offsets = _offsets(case, seed).tolist() if case["kind"] == "moe" else None
    for layer in range(len(_shapes(case))):
        w = _weights(case, seed, layer)
        x = _activations64(case, _activations(case, seed, layer))
        if offsets is None:
            out.append(x @ _weights64(case, w).t())
            continue
        y = torch.empty((x.shape[0], w.shape[1]), dtype=torch.float64, device="cuda")
        for e in range(case["experts"]):
            if offsets[e + 1] > offsets[e]:
                y[offsets[e]:offsets[e + 1]] = x[offsets[e]:offsets[e + 1]] @ \
                    _weights64(case, w[e]).t()
        out.append(y)
    return out[0] if case["kind"] == "layer" else out
