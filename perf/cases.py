"""Timing cases of the decode-time sparse fully-connected layer: what a program that serves a model calls, over the
range of sizes, token counts, weight types and sparsities that it meets.

A decode step walks over the layers of a model and comes back to a layer only after all the others, and a serving
loop records such a step into a HIP graph once and replays it with new inputs.  A case with ``launch: "graph"``
therefore runs a few layers of one shape, each with weights of its own (together more than the last-level cache
holds), as one replay.  ``launch: "eager"`` calls the binding directly.

Kinds of work (``op``):

* ``fc``     one layer: centre, threshold, gather, GEMV (``sparse_fc``; ``dense_fc`` where the sparsity is 0);
* ``block``  the fused SwiGLU block K -> F -> N (``swiglu_block``);
* ``layer``  the fully-connected work of one decoder layer: QKV, O and the SwiGLU block;
* ``setup``  what loading a layer costs: calibration of its input, packing of gate and up, the fused bias.

``counts``: the program also watches how many channels each token kept (``nnz_out``).
"""
import math

import torch

import paper_2412_07174_amd as scap

WEIGHT_TYPE = {"bf16": torch.bfloat16, "f16": torch.float16, "i8": torch.int8}
ACT_TYPE = {"bf16": torch.bfloat16, "f16": torch.float16}


def _fc(name, K, N, B, w, s, layers, act="bf16", law="prenorm", launch="graph", counts=False):
    return {"name": name, "op": "fc", "K": K, "N": N, "B": B, "w": w, "act": act, "s": s, "law": law,
            "counts": counts, "layers": layers, "launch": launch}


def _block(name, K, F, N, B, w, s_x, s_z, layers, act="bf16"):
    return {"name": name, "op": "block", "K": K, "F": F, "N": N, "B": B, "w": w, "act": act, "s": s_x, "s_z": s_z,
            "law": "prenorm", "layers": layers, "launch": "graph"}


def listed():
    return [
        # the smallest call: one 1024 -> 4096 layer, called by itself from Python (latency, launches, host work)
        _fc("fc_1024x4096_f16_b1_eager", 1024, 4096, 1, "f16", 0.5, 1, act="f16", law="laplace", launch="eager",
            counts=True),
        # the down projection of a 7B model, one token: at the usual sparsity, and where next to nothing is read
        _fc("down_14336x4096_bf16_b1_s50", 14336, 4096, 1, "bf16", 0.5, 6, law="swiglu"),
        _fc("down_14336x4096_bf16_b1_s90", 14336, 4096, 1, "bf16", 0.9, 16, law="swiglu"),
        # everything fully connected in a decoder layer of that model, one token
        {"name": "layer_4096_bf16_b1_s50", "op": "layer", "K": 4096, "qkv": 6144, "F": 14336, "B": 1, "w": "bf16",
         "act": "bf16", "s": 0.5, "s_z": 0.5, "law": "prenorm", "layers": 2, "launch": "graph"},
        # a much larger model's feed-forward block, one token
        _block("block_8192x28672_bf16_b1_s50", 8192, 28672, 8192, 1, "bf16", 0.5, 0.5, 1),
        # experts of a mixture-of-experts layer, int8, about two tokens each after routing
        _block("experts_4096x14336_i8_b2", 4096, 14336, 4096, 2, "i8", 0.4, 0.7, 4),
        # small decoding batches through a 7B model's feed-forward block
        _block("block_4096x11008_bf16_b4_s50", 4096, 11008, 4096, 4, "bf16", 0.5, 0.5, 2),
        _block("block_4096x14336_bf16_b16_s70", 4096, 14336, 4096, 16, "bf16", 0.7, 0.7, 2),
        # a batch over fp16 weights, whose kept channels are watched, and a larger one over int8 weights: single layers
        _fc("up_4096x11008_f16_b8_s50", 4096, 11008, 8, "f16", 0.5, 5, act="f16", counts=True),
        _fc("down_14336x4096_i8_b12_s70", 14336, 4096, 12, "i8", 0.7, 6, law="swiglu"),
        # a layer whose sizes fit nothing: odd input length, columns that end inside a tile, three tokens, centred inputs
        _fc("ragged_5461x2744_bf16_b3_s60", 5461, 2744, 3, "bf16", 0.6, 12, law="laplace"),
        # load time of a layer: the calibration sample of the paper's size, packing, the fused bias
        {"name": "setup_4096x14336_bf16_n16384", "op": "setup", "n": 16384, "K": 4096, "F": 14336, "w": "bf16",
         "act": "bf16", "s": 0.5, "law": "laplace", "launch": "eager"},
    ]


def _spread(rng, lo, hi, multiple):
    """A size between lo and hi, spread over its logarithm, a multiple of `multiple`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(v / multiple)) * multiple)


def _layers(weight_bytes):
    return max(1, min(16, int(round(400e6 / weight_bytes))))


def draw(rng):
    w = rng.choice(["bf16", "bf16", "f16", "i8"])
    act = "f16" if w == "f16" else "bf16"
    size = 1 if w == "i8" else 2
    col = 16 if w == "i8" else 8
    B = rng.choice([1, 1, 1, 1, 1, 2, 3, 4, rng.randint(5, 16), rng.randint(5, 16)])
    s = round(rng.uniform(0.3, 0.95), 2)
    kind = rng.choice(["fc", "fc", "fc", "fc", "block", "block", "block", "small", "setup"])
    if kind == "fc":
        K = _spread(rng, 1024, 16384, rng.choice([1, 1, 8, 64, 64]))
        N = _spread(rng, 1024, 28672, rng.choice([col, 128]))
        s = rng.choice([0.0, s, s, s, s, s, s, s])
        while K * N * size > 6e8:
            K = (K + 1) // 2
        c = _fc("", K, N, B, w, s, _layers(K * N * size), act=act, law=rng.choice(["prenorm", "swiglu", "laplace"]),
                counts=s > 0 and rng.random() < 0.2)
    elif kind == "block":
        B = min(B, 4) if w == "f16" else B
        K = _spread(rng, 1024, 8192, rng.choice([8, 64, 128]))
        F = _spread(rng, 2048, 24576, rng.choice([8, 64, 256]))
        while 3 * K * F * size > 8e8:
            F = F // 16 * 8
        N = K if K % col == 0 else (K // col + 1) * col
        c = _block("", K, F, N, B, w, s, round(rng.uniform(0.3, 0.95), 2), _layers(3 * K * F * size), act=act)
    elif kind == "small":
        K, N = _spread(rng, 256, 2048, rng.choice([1, 8, 64])), _spread(rng, 512, 4096, col)
        c = _fc("", K, N, B, w, s, 1, act=act, law=rng.choice(["prenorm", "laplace"]), launch="eager",
                counts=rng.random() < 0.5)
    else:
        w = rng.choice(["bf16", "f16"])
        K = _spread(rng, 1024, 8192, 8)
        n, F = _spread(rng, 256, (1 << 26) // K, 1), _spread(rng, 2048, min(14336, 58000000 // K), 8)
        c = {"op": "setup", "n": n, "K": K, "F": F, "w": w, "act": w, "s": s, "law": "laplace", "launch": "eager"}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _inputs(g, rows, K, law, dtype, scale):
    """Activations of the three families of layer inputs (`scale`: the fixed per-channel scale of a normed input)."""
    if law == "prenorm":
        a = torch.randn(rows, K, generator=g, device="cuda") * scale
    elif law == "swiglu":
        a = torch.randn(rows, K, generator=g, device="cuda")
        a = torch.nn.functional.silu(a) * torch.randn(rows, K, generator=g, device="cuda")
    else:
        u = torch.rand(rows, K, generator=g, device="cuda").clamp_(1e-7, 1 - 1e-7) - 0.5
        a = 0.1 - 0.5 * u.sign() * torch.log1p(-2 * u.abs())
    return a.to(dtype)


def _constants(g, K, law, dtype, s, scale):
    """(m, tau) of a layer from a sample of its inputs: median where the mode lies off zero, else 0; the order statistic."""
    v = _inputs(g, 64, K, law, dtype, scale).float().flatten()
    m = float(v.sort().values[v.numel() // 2]) if law == "laplace" else 0.0
    if s <= 0:
        return m, 0.0
    return m, float((v - m).abs().sort().values[max(0, math.ceil(s * v.numel()) - 1)])


def _weights(g, K, N, w):
    """(weights [K, N], column scales or None): N(0, 0.02^2), int8 ones quantised per column."""
    a = torch.randn(K, N, generator=g, device="cuda") * 0.02
    if w != "i8":
        return a.to(WEIGHT_TYPE[w]), None
    scale = (a.abs().amax(0) / 127).half().clamp_(min=6e-8)
    return (a / scale.float()).round_().clamp_(-127, 127).to(torch.int8), scale


def _wide(W, scale):
    return W.double() if scale is None else W.double() * scale.double()


def _gated_threshold(x, keep, Wg, Wu, s_z):
    """Threshold of the gated product, from the products of the block's own inputs; two digits, as a stored constant has."""
    d = torch.where(keep, x, 0.0).float()
    z = torch.nn.functional.silu(d @ Wg) * (d @ Wu)
    v = z.abs().flatten().sort().values
    return float("%.2g" % float(v[max(0, math.ceil(s_z * v.numel()) - 1)]))


def _fc_problem(g, K, N, case, law):
    act = ACT_TYPE[case["act"]]
    scale = torch.rand(K, generator=g, device="cuda") * 1.5 + 0.5
    m, tau = _constants(g, K, law, act, case["s"], scale)
    W, ws = _weights(g, K, N, case["w"])
    x = _inputs(g, case["B"], K, law, act, scale)
    return {"W": W, "scale": ws, "x": x, "m": m, "tau": tau, "dense": case["s"] <= 0}


def _block_problem(g, K, F, N, case):
    act = ACT_TYPE[case["act"]]
    scale = torch.rand(K, generator=g, device="cuda") * 1.5 + 0.5
    _, tau = _constants(g, K, "prenorm", act, case["s"], scale)
    (Wg, sg), (Wu, su), (Wd, sd) = (_weights(g, a, b, case["w"]) for a, b in ((K, F), (K, F), (F, N)))
    x = _inputs(g, case["B"], K, "prenorm", act, scale)
    sample = _inputs(g, 8, K, "prenorm", act, scale)
    f = (lambda W, s: W.float() if s is None else W.float() * s.float())
    tau_z = _gated_threshold(sample, sample.float().abs() > tau, f(Wg, sg), f(Wu, su), case["s_z"])
    return {"Wg": Wg, "sg": sg, "Wu": Wu, "su": su, "Wd": Wd, "sd": sd, "x": x, "tau": tau, "tau_z": tau_z}


def _problems(case, seed):
    """The layers of one pass, as plain tensors and numbers."""
    g = _generator(seed)
    K, op = case["K"], case["op"]
    out = []
    for _ in range(case.get("layers", 1)):
        if op == "fc":
            out.append(("fc", _fc_problem(g, K, case["N"], case, case["law"])))
        elif op == "block":
            out.append(("block", _block_problem(g, K, case["F"], case["N"], case)))
        elif op == "layer":
            out.append(("fc", _fc_problem(g, K, case["qkv"], case, "prenorm")))
            out.append(("fc", _fc_problem(g, K, K, case, "prenorm")))
            out.append(("block", _block_problem(g, K, case["F"], K, case)))
        else:
            gate, _ = _weights(g, K, case["F"], case["w"])
            up, _ = _weights(g, K, case["F"], case["w"])
            bias = torch.randn(2 * case["F"], generator=g, device="cuda") * 0.1
            out.append(("setup", {"X": _inputs(g, case["n"], K, case["law"], ACT_TYPE[case["act"]], None),
                                  "gate": gate, "up": up, "bias": bias}))
    return out


# ------------------------------------------------------------------------------------------------ the pass
def _ready(kind, p, case):
    """What a program keeps for one layer: weights in the library's layout, constants, workspace, output buffers."""
    B = case.get("B", 1)
    if kind == "fc":
        K, N = p["W"].shape
        ws = scap.Workspace(K, N, B)
        b = None
        if p["m"] != 0.0 and not p["dense"]:
            b = scap.fold_bias(p["W"], p["m"], None, col_scale=p["scale"], workspace=ws)
        counts = case.get("counts", False)
        return dict(p, ws=ws, b=b, y=torch.empty(B, N, device="cuda"),
                    nnz=torch.empty(B, dtype=torch.int32, device="cuda") if counts else None)
    if kind == "block":
        K, F = p["Wg"].shape
        N = p["Wd"].shape[1]
        gu = scap.pack_gate_up(p["Wg"], p["Wu"])
        s = None if p["sg"] is None else scap.pack_gate_up(p["sg"], p["su"])
        return {"W_gu": gu, "gu_scale": s, "W_down": p["Wd"], "down_scale": p["sd"], "x": p["x"], "tau": p["tau"],
                "tau_z": p["tau_z"], "ws": scap.Workspace(K, N, B, F=F), "y": torch.empty(B, N, device="cuda")}
    return dict(p, ws=scap.Workspace(p["gate"].shape[0], 2 * p["gate"].shape[1], 1))


def _call(kind, h, case):
    if kind == "fc":
        if h["dense"]:
            return [scap.dense_fc(h["W"], h["x"], None, col_scale=h["scale"], y=h["y"], workspace=h["ws"])]
        y = scap.sparse_fc(h["W"], h["x"], h["m"], h["tau"], h["b"], col_scale=h["scale"], y=h["y"], nnz_out=h["nnz"],
                           workspace=h["ws"])
        return [y] if h["nnz"] is None else [y, h["nnz"]]
    if kind == "block":
        return [scap.swiglu_block(h["W_gu"], h["W_down"], h["x"], 0.0, h["tau"], None, 0.0, h["tau_z"], None,
                                  gu_scale=h["gu_scale"], down_scale=h["down_scale"], y=h["y"], workspace=h["ws"])]
    m, tau = scap.calibrate(h["X"], case["s"], scap.MODE_MEDIAN, workspace=h["ws"])
    W = scap.pack_gate_up(h["gate"], h["up"])
    return [m, tau, W, scap.fold_bias(W, m, h["bias"], workspace=h["ws"])]


def prepare(case, seed):
    work = [(kind, _ready(kind, p, case)) for kind, p in _problems(case, seed)]
    state = {"case": case, "work": work, "graph": None}
    if case["launch"] == "graph":
        for kind, h in work:  # once by itself: a recording loads no kernels
            _call(kind, h, case)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            state["out"] = [_call(kind, h, case) for kind, h in work]
    torch.cuda.synchronize()
    return state


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return state["out"]
    return [_call(kind, h, state["case"]) for kind, h in state["work"]]


# ------------------------------------------------------------------------------------------------ what it comes to
def _normal_below(t):
    return math.erf(t / math.sqrt(2))


def _union(case, law, s, B):
    """Share of the rows that at least one of B tokens keeps."""
    if s <= 0:
        return 1.0
    if law != "prenorm":
        return 1 - s ** B
    c = [0.5 + 1.5 * (i + 0.5) / 200 for i in range(200)]  # a normed input's channels have scales of their own
    lo, hi = 0.0, 10.0
    for _ in range(50):
        t = (lo + hi) / 2
        lo, hi = (t, hi) if sum(_normal_below(t / v) for v in c) / len(c) < s else (lo, t)
    return 1 - sum(_normal_below(lo / v) ** B for v in c) / len(c)


def work(case):
    size = 1 if case["w"] == "i8" else 2
    B = case.get("B", 1)

    def fc(K, N, s, law, x_bytes=2):
        rows = _union(case, law, s, B) * K
        return rows * N * size + B * K * x_bytes + B * N * 4, 2.0 * B * (1 - s) * K * N

    if case["op"] == "setup":
        n, K, F = case["n"], case["K"], case["F"]
        return {"bytes": 2.0 * n * K + 2 * (2 * K * F * 2) + 2 * K * F * 2 + 16 * F, "flops": 2.0 * K * F}
    parts = []
    if case["op"] == "layer":
        parts += [fc(case["K"], case["qkv"], case["s"], "prenorm"), fc(case["K"], case["K"], case["s"], "prenorm")]
    if case["op"] in ("layer", "block"):
        N = case.get("N", case["K"])
        up, down = fc(case["K"], 2 * case["F"], case["s"], "prenorm"), fc(case["F"], N, case["s_z"], "swiglu", 0)
        parts += [(up[0] - B * 2 * case["F"] * 4, up[1]), down]
    if case["op"] == "fc":
        parts.append(fc(case["K"], case["N"], case["s"], case["law"]))
    L = case.get("layers", 1)
    return {"bytes": L * sum(p[0] for p in parts), "flops": L * sum(p[1] for p in parts)}


def tolerance(case):
    if case["op"] == "setup":
        return {"rel": 2e-6, "max": 2e-5}
    if case["op"] == "fc":
        # sums of up to 16384 products in 32 bits; from 3 tokens on the centred input travels as two 16-bit halves
        return {"rel": 2e-6, "max": 2e-5} if case["B"] <= 2 else {"rel": 1e-5, "max": 1e-4}
    # a gated product next to its threshold may fall either way when the sums before it are taken in another order
    return {"rel": 1e-2, "max": 0.2}


def exact(case, seed):
    out = []
    for kind, p in _problems(case, seed):
        if kind == "fc":
            d = p["x"].float() if p["dense"] else p["x"].float() - p["m"]
            keep = torch.ones_like(d, dtype=torch.bool) if p["dense"] else d.abs() > p["tau"]
            W = _wide(p["W"], p["scale"])
            y = torch.where(keep, d, 0.0).double() @ W
            if not p["dense"]:
                y += p["m"] * W.sum(0)
            out.append([y, keep.sum(1).int()] if case.get("counts", False) else [y])
        elif kind == "block":
            d = p["x"].float()
            d = torch.where(d.abs() > p["tau"], d, 0.0).double()
            z = torch.nn.functional.silu(d @ _wide(p["Wg"], p["sg"])) * (d @ _wide(p["Wu"], p["su"]))
            out.append([torch.where(z.abs() > p["tau_z"], z, 0.0) @ _wide(p["Wd"], p["sd"])])
        else:
            v = p["X"].float().flatten().sort().values
            h = v.numel() // 2
            m = float((v[h].double() + v[(v.numel() - 1) // 2].double()) / 2)
            m = float(torch.tensor(m, dtype=torch.float32))
            tau = float((v - m).abs().sort().values[max(0, math.ceil(case["s"] * v.numel()) - 1)])
            rows, F = p["gate"].shape
            W = torch.stack([p["gate"].view(rows, F // 4, 4), p["up"].view(rows, F // 4, 4)], 2).reshape(rows, 2 * F)
            out.append([m, tau, W, p["bias"].double() + m * W.double().sum(0)])
    return out
