"""What is timed: the linear layers of the Llama shapes this repository serves,
called the way a serving engine calls them.

Two kinds of case:

* "block": the seven linear modules of a transformer block (several blocks in
  a row with `blocks` > 1, each with weights of its own): q, k, v as one
  grouped call; o with the post-EC tail (residual and RMSNorm); gate, up as one
  grouped call; down with the tail. Each call has an input of its own (attention
  and the activation between them are not part of the layer), so every output
  is one layer away from its input. A decode step is captured once as a HIP
  graph and replayed, as an engine does; prefill chunks are called eagerly,
  since their sizes change from step to step.
* "linear": one module, called eagerly through the binding.

Shapes are the Llama-3.2-1B, Llama-3-8B and Llama-2-70B layers of
paper_2606_11244_amd.synth, the 70B layers' shard on one of eight GPUs, and
generic ones. Weights are N(0, 0.02) quantised round-to-nearest, activations
N(0, 1) with 1% of the channels x 20 at prefill, EC factors N(0, 0.01).
"""
import math

import torch

from paper_2606_11244_amd import spear as sp
from paper_2606_11244_amd import synth

_MODULES = ("q", "k", "v", "o", "gate", "up", "down")
_DT = {"f16": torch.float16, "bf16": torch.bfloat16}
_CODE = {"f16": sp.F16, "bf16": sp.BF16}
_GATE = {"one": sp.GATE_ONE, "sigmoid": sp.GATE_SIGMOID_LINEAR, "tanh": sp.GATE_TANH_MLP}
_EPS = 1e-5


def _tp8(shapes):
    """One of eight tensor-parallel shards: column-parallel modules split N,
    row-parallel ones (o, down) split K."""
    return {m: (k // 8, n) if m in ("o", "down") else (k, n // 8) for m, (k, n) in shapes.items()}


_SHAPES = {"1b": synth.LLAMA_1B, "8b": synth.LLAMA_8B, "70b": synth.LLAMA_70B,
           "70b/8": _tp8(synth.LLAMA_70B)}


def _block(name, model, M, *, blocks=1, dtype="f16", group=128, rank=16, gate="sigmoid",
           ec="all", int8=False, bits=4, graph=None):
    c = dict(kind="block", model=model, M=M, blocks=blocks, dtype=dtype, group=group, rank=rank,
             gate=gate, ec=ec, int8=int8, bits=bits, graph=M <= 64 if graph is None else graph)
    return dict(c, name=name) if name else c


def _linear(name, M, N, K, *, dtype="f16", group=128, rank=16, gate="sigmoid", ec=True,
            int8=False, bits=4):
    c = dict(kind="linear", M=M, N=N, K=K, dtype=dtype, group=group, rank=rank, gate=gate, ec=ec,
             int8=int8, bits=bits)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one token through one small projection, called eagerly: nothing but latency
        _linear("call 1b k, 1 token", 1, 512, 2048),
        # interactive decode of one sequence on the small model, four blocks of its graph
        _block("1b decode 1", "1b", 1, blocks=4),
        # a small model serving 24 sequences, INT8 factors (the deployed format)
        _block("1b decode 24, int8", "1b", 24, blocks=4, int8=True),
        # the 8B configuration: bf16, per-channel scales, rank 32, the paper's tanh-MLP gate
        _block("8b decode 8, tanh", "8b", 8, dtype="bf16", group=0, rank=32, gate="tanh"),
        # the headline model at one token, the EC on a quarter of the modules
        _block("70b decode 1", "70b", 1, rank=64, ec="q,gate"),
        # 3-bit backbone, four sequences
        _block("70b w3 decode 4", "70b", 4, rank=64, ec="v,up", bits=3),
        # one of eight tensor-parallel shards serving 16 sequences
        _block("70b/8 decode 16", "70b/8", 16, rank=64),
        # a busy decode batch on the headline model
        _block("70b decode 48", "70b", 48, rank=64, ec="k,o,down"),
        # a ragged chunk through a layer of no particular shape
        _linear("ragged 77", 77, 5000, 2944, dtype="bf16", rank=24),
        # a chunk as the latency-bound scheduler cuts it, 8B
        _block("8b chunk 300", "8b", 300, dtype="bf16", group=0, rank=32),
        # a long prompt on the small model
        _block("1b prefill 2048", "1b", 2048),
        # a long prompt on the headline model
        _block("70b prefill 4096", "70b", 4096, rank=64, ec="q,gate"),
    ]


def draw(rng):
    M = int(round(math.exp(rng.uniform(0.0, math.log(4096.0)))))
    opt = dict(dtype=rng.choice(("f16", "bf16")), group=rng.choice((128, 128, 0)),
               gate=rng.choice(("sigmoid", "sigmoid", "sigmoid", "tanh", "one")),
               int8=rng.random() < 0.25, bits=3 if rng.random() < 0.15 else 4)
    if rng.random() < 0.3:
        N = int(round(math.exp(rng.uniform(math.log(200.0), math.log(16000.0)))))
        K = 128 * int(round(math.exp(rng.uniform(math.log(4.0), math.log(128.0)))))
        return _linear(None, M, N, K, rank=rng.choice((4, 8, 16, 24, 32, 64)), ec=rng.random() < 0.8,
                       **opt)
    model = rng.choice(("1b", "8b", "70b", "70b/8"))
    rank = {"1b": 16, "8b": 32}.get(model, 64)
    some = ",".join(m for m in _MODULES if rng.random() < 0.3)
    return _block(None, model, M, blocks=rng.choice((1, 2, 4)) if model == "1b" and M <= 64 else 1,
                  rank=rank, ec=rng.choice(("all", some)), **opt)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _modules(case):
    """(name, N, K, with EC) of every module of a case, in call order."""
    if case["kind"] == "linear":
        return [("linear", case["N"], case["K"], bool(case["ec"]))]
    on = _MODULES if case["ec"] == "all" else tuple(case["ec"].split(","))
    return [(m, n, k, m in on) for _ in range(case["blocks"])
            for m, (k, n) in ((m, _SHAPES[case["model"]][m]) for m in _MODULES)]


def _generator(seed, *ids):
    g = torch.Generator(device="cuda")
    s = seed % (1 << 40)
    for i in ids:
        s = s * 1009 + i + 1
    g.manual_seed(s % (1 << 62))
    return g


def _randn(shape, g, std=1.0):
    return torch.randn(shape, device="cuda", generator=g) * std


def _int8_rows(w):
    s = w.abs().amax(dim=1) / 127.0
    s = torch.where(s > 0, s, torch.ones_like(s))
    return torch.clamp(torch.round(w / s[:, None]), -127, 127).to(torch.int8), s.float()


def _weights(case, seed, i, N, K, with_ec):
    """One module's stored values: codes [N][K] (not yet packed), scales, zero
    points and, with an EC, its factors and gate."""
    g = _generator(seed, 1, i)
    G = K if case["group"] == 0 else case["group"]
    top = float((1 << case["bits"]) - 1)
    q = torch.empty((N, K), dtype=torch.uint8, device="cuda")
    s = torch.empty((N, K // G), dtype=torch.float16, device="cuda")
    z = torch.empty((N, K // G), dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 26) // K)
    for r0 in range(0, N, step):
        w = _randn((min(step, N - r0), K // G, G), g, 0.02)
        lo, hi = w.amin(dim=2), w.amax(dim=2)
        sh = ((hi - lo) / top).half()
        zf = torch.clamp(torch.round(-lo / sh.float()), 0, top)
        qf = torch.clamp(torch.round(w / sh.float()[:, :, None]) + zf[:, :, None], 0, top)
        q[r0:r0 + step] = qf.to(torch.uint8).reshape(-1, K)
        s[r0:r0 + step] = sh
        z[r0:r0 + step] = zf.to(torch.uint8)
    ec = None
    if with_ec:
        r, dt = case["rank"], _DT[case["dtype"]]
        A, B = _randn((r, K), g, 0.01), _randn((N, r), g, 0.01)
        ec = dict(b_g=0.1, alpha=1.0)
        if case["int8"]:
            ec["A"], ec["a_scale"] = _int8_rows(A)
            ec["B"], ec["b_scale"] = _int8_rows(B)
        else:
            ec["A"], ec["B"] = A.to(dt), B.to(dt)
        if case["gate"] == "sigmoid":
            ec["w_g"] = _randn((K,), g, 0.05).to(dt)
        if case["gate"] == "tanh":
            h = 4 * r
            ec["W1"], ec["b1"] = _randn((h, r), g, r ** -0.5).to(dt), _randn((h,), g, 0.1).to(dt)
            ec["W2"], ec["b2"] = _randn((r, h), g, h ** -0.5).to(dt), _randn((r,), g, 0.1).to(dt)
    return q, s, z, ec


def _input(case, seed, i, K):
    g = _generator(seed, 2, i)
    x = _randn((case["M"], K), g)
    if case["M"] > 64:  # prefill: outlier channels
        idx = torch.randperm(K, device="cuda", generator=g)[: round(0.01 * K)]
        x[:, idx] *= 20.0
    return x.to(_DT[case["dtype"]])


def _tail(case, seed, i, N):
    g = _generator(seed, 3, i)
    dt = _DT[case["dtype"]]
    return _randn((case["M"], N), g).to(dt), (1.0 + _randn((N,), g, 0.1)).to(dt)


def _pack(q, bits):
    """Codes to the words of include/spear.h."""
    N, K = q.shape
    if bits == 4:
        return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous().view(torch.int32)
    out = torch.empty((N, K // 32, 3), dtype=torch.int32, device=q.device)
    step = max(1, (1 << 25) // K)
    sh = torch.arange(8, device=q.device, dtype=torch.int64)
    for r0 in range(0, N, step):
        c = q[r0:r0 + step].to(torch.int64).view(-1, K // 32, 16, 2)
        e, o = c[..., 0], c[..., 1]
        low = [((e[..., 8 * h:8 * h + 8] & 3) << (2 * sh)).sum(-1)
               | (((o[..., 8 * h:8 * h + 8] & 3) << (2 * sh + 16)).sum(-1)) for h in (0, 1)]
        s16 = torch.arange(16, device=q.device, dtype=torch.int64)
        high = ((e >> 2) << s16).sum(-1) | ((o >> 2) << (s16 + 16)).sum(-1)
        w = torch.stack((low[0], low[1], high), dim=-1)
        out[r0:r0 + step] = torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)
    return out.view(N, K // 32 * 3)


def _problem(case, N, K, with_ec):
    return sp.problem(case["M"], N, K, case["group"], _CODE[case["dtype"]],
                      case["rank"] if with_ec else 0, _GATE[case["gate"]], 0, sp.PATH_AUTO, case["bits"])


def _shared_input(case, i):
    """The module whose input module i reads (k, v read q's; up reads gate's)."""
    if case["kind"] == "linear":
        return i
    b, j = divmod(i, 7)
    return 7 * b + (0, 0, 0, 3, 4, 4, 6)[j]


def prepare(case, seed):
    M, dt = case["M"], _DT[case["dtype"]]
    mods, xs = [], {}
    for i, (name, N, K, with_ec) in enumerate(_modules(case)):
        q, s, z, ec = _weights(case, seed, i, N, K, with_ec)
        xi = _shared_input(case, i)
        if xi not in xs:
            xs[xi] = _input(case, seed, xi, K)
        m = dict(name=name, prob=_problem(case, N, K, with_ec), x=xs[xi],
                 qweight=_pack(q, case["bits"]), scales=s.view(torch.int16), zeros=z, ec_args=ec,
                 y=torch.empty((M, N), dtype=dt, device="cuda"))
        if name in ("o", "down"):
            m["residual"], m["norm_w"] = _tail(case, seed, i, N)
            m["y_norm"] = torch.empty((M, N), dtype=dt, device="cuda")
        mods.append(m)
    blocks = [mods[b:b + 7] for b in range(0, len(mods), 7)]
    need = 256
    for b in blocks:
        for m in b:
            need = max(need, sp.dispatch_plan(m["prob"], m["ec_args"] is not None).workspace_bytes)
        if case["kind"] == "block":
            need = max(need, sp.group_workspace(b[0:3]), sp.group_workspace(b[4:6]))
    st = dict(case=case, blocks=blocks, ws=torch.zeros(need, dtype=torch.uint8, device="cuda"))
    if case.get("graph"):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _call(st)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            st["out"] = _call(st)
        st["graph"] = graph
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _call(st):
    ws, out = st["ws"], []
    if st["case"]["kind"] == "linear":
        m = st["blocks"][0][0]
        a = (m["prob"], m["x"], m["qweight"], m["scales"], m["zeros"])
        if m["ec_args"] is None:
            sp.w4_linear(*a, m["y"], workspace=ws)
        else:
            e = dict(m["ec_args"])
            sp.w4ec_linear(*a, e.pop("A"), e.pop("B"), m["y"], workspace=ws, **e)
        return [m["y"]]

    def tail(m):
        sp.w4ec_linear_tail(m["prob"], m["x"], m["qweight"], m["scales"], m["zeros"], m["y"],
                            ec_args=m["ec_args"], residual=m["residual"], norm_w=m["norm_w"],
                            eps=_EPS, y_norm=m["y_norm"], workspace=ws)

    for q, k, v, o, gate, up, down in st["blocks"]:
        sp.w4ec_linear_group([q, k, v], ws)
        tail(o)
        sp.w4ec_linear_group([gate, up], ws)
        tail(down)
        out += [q["y"], k["y"], v["y"], o["y"], o["y_norm"], gate["y"], up["y"], down["y"],
                down["y_norm"]]
    return out


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return _call(state)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it should give
# ---------------------------------------------------------------------------

def work(case):
    M, b, f = case["M"], 0, 0
    for i, (name, N, K, with_ec) in enumerate(_modules(case)):
        G = K if case["group"] == 0 else case["group"]
        b += N * K * case["bits"] // 8 + 3 * N * (K // G) + 2 * M * N
        f += 2 * M * N * K
        if _shared_input(case, i) == i:
            b += 2 * M * K
        if name in ("o", "down"):
            b += 2 * M * N + 2 * N + 2 * M * N
            f += 6 * M * N
        if with_ec:
            r, w = case["rank"], 1 if case["int8"] else 2
            b += w * r * (N + K) + (4 * (r + N) if case["int8"] else 0)
            f += 2 * M * r * (N + K)
            if case["gate"] == "sigmoid":
                b += 2 * K
                f += 2 * M * K
            if case["gate"] == "tanh":
                b += 2 * (8 * r * r + 5 * r)
                f += 16 * M * r * r
    return {"bytes": b, "flops": f}


def tolerance(case):
    # one rounding of the output and, where a path dequantises the weights to
    # the activation dtype, one of each weight
    return {"rel": 1.6e-3, "max": 1e-2} if case["dtype"] == "f16" else {"rel": 1.2e-2, "max": 8e-2}


def _exact_layer(case, x, q, s, z, ec):
    N, K = q.shape
    G = K if case["group"] == 0 else case["group"]
    x = x.double()
    w = (q.view(N, K // G, G).double() - z.double()[:, :, None]) * s.double()[:, :, None]
    y = x @ w.view(N, K).T
    del w
    if ec is None:
        return y
    A, B = ec["A"].double(), ec["B"].double()
    if "a_scale" in ec:
        A, B = A * ec["a_scale"].double()[:, None], B * ec["b_scale"].double()[:, None]
    u = x @ A.T
    if case["gate"] == "sigmoid":
        u = u * torch.sigmoid(x @ ec["w_g"].double() + ec["b_g"])[:, None]
    elif case["gate"] == "tanh":
        hid = torch.relu(u @ ec["W1"].double().T + ec["b1"].double())
        u = u * (1.0 + torch.tanh(hid @ ec["W2"].double().T + ec["b2"].double()))
    return y + ec["alpha"] * (u @ B.T)


def exact(case, seed):
    out, xs = [], {}
    for i, (name, N, K, with_ec) in enumerate(_modules(case)):
        xi = _shared_input(case, i)
        if xi not in xs:
            xs = {xi: _input(case, seed, xi, K)}
        y = _exact_layer(case, xs[xi], *_weights(case, seed, i, N, K, with_ec))
        if name in ("o", "down"):
            res, nw = _tail(case, seed, i, N)
            y = y + res.double()
            out += [y, y / torch.sqrt((y * y).mean(dim=1, keepdim=True) + _EPS) * nw.double()]
        else:
            out.append(y)
    return out
