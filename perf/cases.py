"""The work that users of this library have it do, as cases that can be timed and compared.

Every case goes through the public calls of ``paper_2511_10645_amd`` the way a program that serves or converts a
model calls them.  Plans, repacked weights, workspaces and (for decode) captured HIP graphs belong to such a
program and are made once by ``prepare``; ``run`` is one pass.  Kinds of cases:

  linears    the rotated W4A16 linears of decoder layers (``paro_rotated_linear``) one after the other, or the bare
             ones (``paro_w4a16_linear``) where the caller transforms the activations itself
  own        projections that share their input, each with its own transform (``paro_rotated_linear_multi``)
  transform  the transform of activations alone (``paro_rotate_scale``), in front of a caller's own product
  mxfp4      the weight-activation linears with both operands in MXFP4 (``paro_rotated_linear_mxfp4``)
  quantize   the weight side, offline: transform and quantise a dense weight (``paro_w4_quantize`` or
             ``paro_mxfp4_quantize_weight``)

Layer shapes are those of ``paro_inputs.CONFIGS`` (an 8B-class and a 32B-class decoder layer, a tiny linear); the
distributions are the ones documented there, drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_2511_10645_amd as paro

MODELS = {
    "tiny": ((512, 512),),
    "8b": ((4096, 6144), (4096, 4096), (4096, 28672), (14336, 4096)),
    "32b": ((5120, 7168), (5120, 5120), (5120, 55296), (27648, 5120)),
}
GROUP, LAYERS, PAIRS = 128, 8, 64
MOST_FLOPS = 3.0e12                 # of a drawn case; the largest listed one has 4.0e12


def listed():
    return [
        # the smallest call there is: one token through one small linear, called eagerly (latency of a call)
        {"name": "tiny_t1", "kind": "linears", "model": "tiny", "copies": 1, "tokens": 1, "graph": False, "bias": False, "transform": True},
        # batch-1 decode: the linears of four decoder layers per captured step, every weight read once
        {"name": "layers8b_t1", "kind": "linears", "model": "8b", "copies": 4, "tokens": 1, "graph": True, "bias": False, "transform": True},
        # batched decode, 16 sequences
        {"name": "layers8b_t16", "kind": "linears", "model": "8b", "copies": 4, "tokens": 16, "graph": True, "bias": False, "transform": True},
        # batched decode of a loaded server, 64 sequences
        {"name": "layers8b_t64", "kind": "linears", "model": "8b", "copies": 4, "tokens": 64, "graph": True, "bias": False, "transform": True},
        # a ragged chunk: short prompt, or decode tokens and a prefill chunk in one batch; biased linears
        {"name": "layer8b_t201", "kind": "linears", "model": "8b", "copies": 2, "tokens": 201, "graph": False, "bias": True, "transform": True},
        # prefill of a 2048-token prompt
        {"name": "layer8b_t2048", "kind": "linears", "model": "8b", "copies": 1, "tokens": 2048, "graph": False, "bias": False, "transform": True},
        # the largest: a 32B-class layer, 4096 prompt tokens
        {"name": "layer32b_t4096", "kind": "linears", "model": "32b", "copies": 1, "tokens": 4096, "graph": False, "bias": False, "transform": True},
        # speculative or small-batch decode with one transform per projection: q / k / v, then gate / up
        {"name": "own8b_t3", "kind": "own", "c_in": 4096, "outs": "4096,1024,1024;14336,14336", "copies": 4, "tokens": 3, "graph": True},
        # an input width that is a multiple of the group but not of 512 (11008 is a common MLP width): such weights
        # stay in the interchange layout
        {"name": "width11008_t24", "kind": "linears", "model": "", "c_in": 11008, "c_out": 4096, "copies": 2, "tokens": 24, "graph": False,
         "bias": False, "transform": True},
        # the transform alone over an odd number of tokens, MLP width
        {"name": "transform_t1023", "kind": "transform", "c_in": 14336, "tokens": 1023, "layers": 8, "scale_order": 0},
        # prefill with 4-bit weights and 4-bit activations
        {"name": "mxfp4_8b_t2048", "kind": "mxfp4", "model": "8b", "copies": 1, "tokens": 2048, "graph": False},
        # converting a model: one MLP weight, transformed and quantised
        {"name": "quantize_gate_up", "kind": "quantize", "c_in": 4096, "c_out": 28672, "format": "int4", "transform": True},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _tokens(rng, most):
    return max(1, min(most, int(round(_log(rng, 1, most)))))


def draw(rng):
    kind = rng.choices(("linears", "own", "transform", "mxfp4", "quantize"), (55, 10, 12, 13, 10))[0]
    if kind == "transform":
        return {"kind": kind, "c_in": GROUP * int(_log(rng, 4, 216)), "tokens": _tokens(rng, 4096), "layers": rng.choice((8, 8, 8, 4)),
                "scale_order": rng.choice((0, 0, 1))}
    c_in = 512 * max(1, min(54, int(round(_log(rng, 1, 54)))))
    c_out = 16 * max(32, int(_log(rng, 32, 3456)))
    while c_in * c_out > 290_000_000:
        c_out = 16 * max(32, int(_log(rng, 32, 3456)))
    if kind == "quantize":
        return {"kind": kind, "c_in": c_in, "c_out": c_out, "format": rng.choice(("int4", "int4", "mxfp4")), "transform": rng.random() < 0.8}
    if kind == "own":
        c_in = min(c_in, 8192)
        outs = ",".join(str(16 * int(_log(rng, 32, 900))) for _ in range(rng.randint(2, 4)))
        return {"kind": kind, "c_in": c_in, "outs": outs, "copies": 4, "tokens": rng.randint(1, 4), "graph": True}
    tokens = _tokens(rng, min(4096, int(MOST_FLOPS / (2.0 * c_in * c_out))))
    copies = max(1, min(8, int(256e6 / (c_in * c_out)))) if tokens <= 512 else 1
    if kind == "linears" and rng.random() < 0.12:         # a width that no whole number of 512-channel slices makes
        c_in += GROUP * rng.randint(1, 3)
        tokens = min(tokens, 48)
    graph = tokens <= 64 and rng.random() < 0.8
    case = {"kind": kind, "model": "", "c_in": c_in, "c_out": c_out, "copies": copies, "tokens": tokens, "graph": graph}
    if kind == "linears":
        case.update(bias=rng.random() < 0.3, transform=rng.random() < 0.85)
    return case


# ---- inputs -------------------------------------------------------------------------------------------------------

def _gen(seed, index):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1009 + index) % (1 << 62))


def _shapes(case):
    return MODELS[case["model"]] if case.get("model") else ((case["c_in"], case["c_out"]),)


def _draw_x(g, tokens, c):
    x = torch.randn((tokens, c), generator=g, device="cuda", dtype=torch.float32)
    hot = torch.randperm(c, generator=g, device="cuda")[:max(1, round(0.005 * c))]
    x[:, hot] *= 50.0                                     # outlier channels
    return x.half()


def _draw_rotation(g, c, layers=LAYERS):
    n = c // GROUP
    pairs = torch.rand((n, layers, GROUP), generator=g, device="cuda").argsort(-1).reshape(n, layers, PAIRS, 2).to(torch.int16)
    theta = (torch.rand((n, layers, PAIRS), generator=g, device="cuda") * 2 - 1) * math.pi
    scale = torch.exp(0.3 * torch.randn(c, generator=g, device="cuda")).half()
    return pairs, theta, scale


def _words(g, shape):
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=g, device="cuda", dtype=torch.int32)


def _draw_w4(g, c, n, bias):
    qweight = _words(g, (n, c // 8))
    scales = (0.005 + 0.015 * torch.rand((c // GROUP, n), generator=g, device="cuda")).half()
    qzeros = _words(g, (c // GROUP, n // 8))
    return qweight, scales, qzeros, (torch.randn(n, generator=g, device="cuda").half() if bias else None)


def _draw_mxfp4(g, c, n):
    return _words(g, (n, c // 8)), torch.randint(116, 122, (n, c // 32), generator=g, device="cuda", dtype=torch.uint8)


def _draw_dense(g, c, n):
    w = torch.randn((n, c), generator=g, device="cuda", dtype=torch.float16)
    w *= 0.02
    rows = torch.arange(n, device="cuda")
    for _ in range(max(1, round(0.005 * c))):             # isolated large weights, as pre-trained weights have them
        w[rows, torch.randint(0, c, (n,), generator=g, device="cuda")] *= 20.0
    return w


def _draws(case, seed):
    """The plain tensors of every call of a pass, in order."""
    kind, copies = case["kind"], case.get("copies", 1)
    if kind in ("linears", "mxfp4"):
        for k in range(copies):
            for j, (c, n) in enumerate(_shapes(case)):
                g = _gen(seed, 16 * k + j)
                d = {"c": c, "n": n, "x": _draw_x(g, case["tokens"], c), "rot": _draw_rotation(g, c)}
                d["w"] = _draw_w4(g, c, n, case["bias"]) if kind == "linears" else _draw_mxfp4(g, c, n)
                yield d
    elif kind == "own":
        for k in range(copies):
            for j, outs in enumerate(case["outs"].split(";")):
                g = _gen(seed, 16 * k + j)
                c = case["c_in"]
                yield {"c": c, "x": _draw_x(g, case["tokens"], c),
                       "parts": [(_draw_rotation(g, c), _draw_w4(g, c, int(n), False)) for n in outs.split(",")]}
    elif kind == "transform":
        g = _gen(seed, 0)
        yield {"c": case["c_in"], "x": _draw_x(g, case["tokens"], case["c_in"]), "rot": _draw_rotation(g, case["c_in"], case["layers"])}
    else:
        g = _gen(seed, 0)
        yield {"c": case["c_in"], "n": case["c_out"], "w": _draw_dense(g, case["c_in"], case["c_out"]),
               "rot": _draw_rotation(g, case["c_in"]) if case["transform"] else None}


# ---- what a program keeps -----------------------------------------------------------------------------------------

def _rotation(rot, scale_order=0):
    pairs, theta, scale = (t.cpu().numpy() for t in rot)
    r = paro.Rotation(pairs, theta, scale, scale_order=scale_order)
    paro.paro_rotation_plan_build(r)
    return r


def _w4(w):
    qweight, scales, qzeros, bias = w
    weight = paro.W4Weight.from_device(qweight, scales, qzeros, bias)
    if weight.c_in % 512 == 0:                            # other widths have no repacked form
        paro.paro_w4_repack(weight)
        weight.drop_interchange()
    return weight


def prepare(case, seed):
    kind, tokens = case["kind"], case.get("tokens", 0)
    calls = []
    if kind == "quantize":
        d = next(iter(_draws(case, seed)))
        rot = _rotation(d["rot"]) if d["rot"] is not None else None
        call = paro.paro_w4_quantize if case["format"] == "int4" else paro.paro_mxfp4_quantize_weight
        return {"kind": kind, "call": call, "rot": rot, "w": d["w"], "int4": case["format"] == "int4"}
    if kind == "transform":
        d = next(iter(_draws(case, seed)))
        return {"kind": kind, "rot": _rotation(d["rot"], case["scale_order"]), "x": d["x"]}
    for d in _draws(case, seed):
        if kind == "linears":
            rot = _rotation(d["rot"]) if case["transform"] else None
            calls.append({"rot": rot, "w": _w4(d["w"]), "x": d["x"]})
        elif kind == "mxfp4":
            weight = paro.Mxfp4Weight(*d["w"])
            paro.paro_mxfp4_repack(weight)
            calls.append({"rot": _rotation(d["rot"]), "w": weight, "x": d["x"]})
        else:
            rots, weights = [_rotation(r) for r, _ in d["parts"]], [_w4(w) for _, w in d["parts"]]
            calls.append({"rots": rots, "ws": weights, "x": d["x"]})
    if kind == "linears":
        work = paro.Workspace.shared([(k["rot"], k["w"], tokens) for k in calls])
    elif kind == "mxfp4":
        work = torch.empty(max(paro.paro_workspace_bytes_mxfp4(k["w"].c_in, tokens) for k in calls), dtype=torch.uint8, device="cuda")
    else:
        total = [paro.paro_workspace_bytes_multi(k["rots"], k["ws"], tokens) for k in calls]
        part = [paro.paro_workspace_exchange_bytes_multi(k["rots"], k["ws"], tokens) for k in calls]
        work = paro.Workspace(max(part) + max(t - p for t, p in zip(total, part)))
    state = {"kind": kind, "calls": calls, "work": work, "graph": None}
    if case["graph"]:                                     # a decode step is captured once and replayed
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _pass(state)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            state["out"] = _pass(state)
        state["graph"] = graph
    return state


def _pass(state):
    kind, work, outs = state["kind"], state["work"], []
    for k in state["calls"]:
        if kind == "mxfp4":
            outs.append(paro.paro_rotated_linear_mxfp4(k["rot"], k["w"], k["x"], work))
        elif kind == "own":
            outs += paro.paro_rotated_linear_multi(k["rots"], k["ws"], k["x"], work)
        elif k["rot"] is not None:
            outs.append(paro.paro_rotated_linear(k["rot"], k["w"], k["x"], work))
        else:
            outs.append(paro.paro_w4a16_linear(k["w"], k["x"], work))
    return outs


def run(state):
    if state["kind"] == "quantize":
        w = state["call"](state["rot"], state["w"])
        return [w.qweight, w.scales, w.qzeros] if state["int4"] else [w.codes, w.scales]
    if state["kind"] == "transform":
        return paro.paro_rotate_scale(state["rot"], state["x"])
    if state["graph"] is not None:
        state["graph"].replay()
        return state["out"]
    return _pass(state)


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def _rotation_bytes(c, layers=LAYERS):
    return c // GROUP * layers * PAIRS * 8 + 2 * c        # pair indices and angle per pair, channel scales


def work(case):
    kind, t = case["kind"], case.get("tokens", 0)
    nbytes = flops = 0
    if kind == "transform":
        c = case["c_in"]
        return {"bytes": 4 * t * c + _rotation_bytes(c, case["layers"]), "flops": 3 * case["layers"] * t * c + t * c}
    if kind == "quantize":
        c, n = case["c_in"], case["c_out"]
        out = n * c // 2 + (n * (c // GROUP) * 5 // 2 if case["format"] == "int4" else n * c // 32)
        return {"bytes": 2 * n * c + out + (_rotation_bytes(c) if case["transform"] else 0),
                "flops": (3 * LAYERS + 1) * n * c if case["transform"] else n * c}
    if kind == "own":
        c = case["c_in"]
        for outs in case["outs"].split(";"):
            nbytes += 2 * t * c
            for n in map(int, outs.split(",")):
                nbytes += n * c // 2 + n * (c // GROUP) * 5 // 2 + 2 * t * n + _rotation_bytes(c)
                flops += 2 * t * n * c + 3 * LAYERS * t * c
        return {"bytes": case["copies"] * nbytes, "flops": case["copies"] * flops}
    for c, n in _shapes(case):
        nbytes += n * c // 2 + (n * (c // GROUP) * 5 // 2 if kind == "linears" else n * c // 32) + 2 * t * (c + n)
        flops += 2 * t * n * c
        if kind == "mxfp4" or case["transform"]:
            nbytes += _rotation_bytes(c)
            flops += 3 * LAYERS * t * c
        if case.get("bias"):
            nbytes += 2 * n
    return {"bytes": case["copies"] * nbytes, "flops": case["copies"] * flops}


def tolerance(case):
    # Four times what a pass is off from exact(): outputs in fp16 from fp32 sums over fp16 operands (transformed
    # activations and, for many tokens, dequantised weights are rounded to fp16): 2.1e-4 to 4.1e-4 in the 2-norm.
    # max: over the larger of a value and the outputs' root mean square.
    if case["kind"] == "transform":
        return {"rel": 8e-4, "max": 2e-3}
    if case["kind"] == "quantize":                        # ties of the rounding to 4 bits (fp32 against fp64 on a CPU: 2e-6 of
        return {"rel": 8e-4, "max": 2e-3, "differ": 1e-4} if case["transform"] else "exact"    # the words, 3e-5 of the scales)
    if case["kind"] == "mxfp4":                           # ties of the activations' rounding to 4 bits, beside the above
        return {"rel": 1.2e-3, "max": 4e-2}
    return {"rel": 1.6e-3, "max": 1e-2}


# ---- the same in 64 bits, from the definitions --------------------------------------------------------------------

def _rotate64(x, rot, scale_order=0, inverse_scale=False):
    pairs, theta, scale = rot
    t, c = x.shape
    s = scale.double().reciprocal() if inverse_scale else scale.double()
    u = x.double()
    if scale_order == 0:
        u = u * s
    u = u.reshape(t, c // GROUP, GROUP)
    for l in range(pairs.shape[1]):
        i = pairs[:, l, :, 0].long().unsqueeze(0).expand(t, -1, -1)
        j = pairs[:, l, :, 1].long().unsqueeze(0).expand(t, -1, -1)
        cos, sin = torch.cos(theta[:, l].double()), torch.sin(theta[:, l].double())
        ui, uj = u.gather(2, i), u.gather(2, j)
        u = u.scatter(2, i, cos * ui - sin * uj).scatter(2, j, sin * ui + cos * uj)
    u = u.reshape(t, c)
    return u * s if scale_order == 1 else u


def _nibbles(words):
    return ((words.unsqueeze(-1) >> torch.arange(0, 32, 4, device=words.device, dtype=torch.int32)) & 15).flatten(-2)


def _linear64(u, w):
    qweight, scales, qzeros, bias = w
    n, outs = qweight.shape[0], []
    for lo in range(0, n, 8192):                          # rows of the weight at a time
        hi = min(n, lo + 8192)
        q = _nibbles(qweight[lo:hi]).double().reshape(hi - lo, -1, GROUP)
        z = _nibbles(qzeros)[:, lo:hi].double().t().unsqueeze(-1)
        d = ((q - z) * scales[:, lo:hi].double().t().unsqueeze(-1)).reshape(hi - lo, -1)
        outs.append(u @ d.t())
    y = torch.cat(outs, 1)
    return y + bias.double() if bias is not None else y


def _e2m1(device):
    return torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device=device)


def _mxfp4_round64(u):
    t, c = u.shape
    v = u.reshape(t, c // 32, 32)
    e = torch.frexp(v.abs().amax(-1, keepdim=True).clamp_min(2.0 ** -125))[1].double() - 1 - 2
    r = v / torch.exp2(e)
    a = r.abs()
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0)).double()
    a = (torch.round(a / step) * step).clamp_max(6.0)     # torch.round: ties to even, which are the even codes
    return (torch.sign(r) * a * torch.exp2(e)).reshape(t, c)


def _mxfp4_linear64(u, w):
    codes, scales = w
    n, outs, table = codes.shape[0], [], _e2m1(codes.device)
    for lo in range(0, n, 8192):
        hi = min(n, lo + 8192)
        d = table[_nibbles(codes[lo:hi]).long()].reshape(hi - lo, -1, 32) * torch.exp2(scales[lo:hi].double() - 127).unsqueeze(-1)
        outs.append(u @ d.reshape(hi - lo, -1).t())
    return torch.cat(outs, 1)


def exact(case, seed):
    kind, outs = case["kind"], []
    for d in _draws(case, seed):
        if kind == "transform":
            return _rotate64(d["x"], d["rot"], case["scale_order"])
        if kind == "quantize":
            if case["format"] != "int4":
                return None
            scales = []
            for lo in range(0, d["n"], 4096):
                w = d["w"][lo:lo + 4096]
                w = _rotate64(w, d["rot"], inverse_scale=True) if d["rot"] is not None else w.double()
                g = w.reshape(w.shape[0], -1, GROUP)
                scales.append(((g.amax(-1) - g.amin(-1)) / 15.0).clamp_min(2.0 ** -14).t())
            return [None, torch.cat(scales, 1), None]
        if kind == "own":
            outs += [_linear64(_rotate64(d["x"], r), w) for r, w in d["parts"]]
        elif kind == "mxfp4":
            outs.append(_mxfp4_linear64(_mxfp4_round64(_rotate64(d["x"], d["rot"])), d["w"]))
        else:
            outs.append(_linear64(_rotate64(d["x"], d["rot"]) if case["transform"] else d["x"].double(), d["w"]))
    return outs
