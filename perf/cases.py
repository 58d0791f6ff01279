"""The work whose speed is measured: what a user of the library has it do.

Sizes are those of the repository's workloads (paper_2402_04925_amd/inputs.py:
the Llama-70B MLP, 8192 x 28672 x 8192, and the Granite-20B MLP, 6144 x 24576 x
6144, at their tensor-parallel degrees) or generic. Every input is drawn on the
GPU from the seed, with the distributions of that module: uniform codes and
zeros, scales in [0.002, 0.02], standard normal activations, act-order by a
random permutation (Eq. 2-3).

A case holds
  op      "gemm" (w4a16_gemm), "mlp" (mlp_shard), "gated" (gated_mlp_shard) or
          "reorder" (the offline reorder of a layer pair)
  path    "ordered" (rows sorted by group) or "actorder" (metadata through g_idx)
  layout  "tiled" or "gptq" storage of the packed weights
  dtype   "fp16" or "bf16" activations, scales and outputs
  M       tokens of the call
  K, N    the first layer as this rank holds it; N2 the second layer's outputs
  tp      tensor-parallel degree: an act-order row shard keeps the whole layer's
          metadata, tp times its own
  G       group size (a partial last group where G does not divide the rows)
  perm    gemm: the call gathers X[:, x_perm] (Alg. 2's local step)
  layers  calls of a pass, one for each layer of a stack, each with weights and
          activations of its own, as one decode step makes them
  graph   the pass is a HIP graph captured once and replayed for each token, as
          a serving loop (and bench.py) runs decode; otherwise each call is made
          from Python
"""
from __future__ import annotations

import math

import torch

import paper_2402_04925_amd as tpdq

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}
PATHS = {"ordered": tpdq.PATH_ORDERED, "actorder": tpdq.PATH_ACTORDER}


def _case(name, op, M, K, N, N2=0, G=128, tp=1, dtype="fp16", path="ordered", layout="tiled", perm=False,
          layers=1, graph=False):
    c = dict(op=op, M=M, K=K, N=N, N2=N2, G=G, tp=tp, dtype=dtype, path=path, layout=layout, perm=perm,
             layers=layers, graph=graph)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: the repository's tiny single GEMM, from Python (launch and host latency)
        _case("gemm_tiny", "gemm", 4, 256, 128, G=32),
        # token generation for one sequence: Llama-70B at TP = 8, a stack of layers per token
        _case("decode_m1", "mlp", 1, 8192, 3584, 8192, tp=8, layers=8, graph=True),
        # token generation for a batch of 16: the repository's headline workload
        _case("decode_m16", "mlp", 16, 8192, 3584, 8192, tp=8, layers=8, graph=True),
        # the same model with its gate projection, bf16, a small batch
        _case("gated_decode_m4", "gated", 4, 8192, 3584, 8192, tp=8, dtype="bf16", layers=4, graph=True),
        # a full serving batch, Granite-20B at TP = 4
        _case("batch_m64", "mlp", 64, 6144, 6144, 6144, tp=4, dtype="bf16", layers=4, graph=True),
        # the same batch on one GPU that holds the whole Llama-70B MLP
        _case("unsharded_m64", "mlp", 64, 8192, 28672, 8192),
        # a short ragged prompt through one layer, with the column gather of Alg. 2; odd sizes, small groups
        _case("gemm_ragged_m77", "gemm", 77, 5000, 3464, G=64, perm=True),
        # prefill of a long prompt, Llama-70B at TP = 2
        _case("prefill_m2048", "mlp", 2048, 8192, 14336, 8192, tp=2),
        # a prompt of 1000 tokens through the gated MLP, TP = 8, bf16
        _case("gated_prefill_m1000", "gated", 1000, 8192, 3584, 8192, tp=8, dtype="bf16"),
        # a checkpoint used without the offline reorder: generation and prompt
        _case("actorder_m16", "mlp", 16, 8192, 3584, 8192, tp=8, path="actorder", layout="gptq", layers=4, graph=True),
        _case("actorder_prefill_m512", "mlp", 512, 6144, 6144, 6144, tp=4, path="actorder", layout="gptq"),
        # loading a model: Alg. 1 and the fold on a whole Llama-70B layer pair
        _case("reorder", "reorder", 0, 8192, 28672, 8192),
    ]


def _log_uniform(rng, lo, hi, step):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    """Another case of the ranges above: 1 to 2048 tokens, layers from 512 to 16384 rows or columns (most of
    them whole tiles, some ragged), both types, all options. Costs are bounded by the largest listed case."""
    op = rng.choices(["mlp", "gated", "gemm", "reorder"], [8, 5, 5, 2])[0]
    dtype = rng.choice(["fp16", "bf16"])
    G = rng.choice([32, 64, 128, 128, 128])
    step = rng.choice([8, 128, 128, 128])  # one in four ragged
    K = _log_uniform(rng, 1024, 8192, step)
    N = _log_uniform(rng, 512, 14336, step)
    N2 = K if op in ("mlp", "gated") else 0
    if op == "reorder":
        return _case(None, op, 0, K, N, K, G=G, dtype=dtype)
    path = rng.choices(["ordered", "actorder"], [4, 1])[0] if op != "gated" else "ordered"
    layout = "tiled" if path == "ordered" else rng.choice(["gptq", "gptq", "tiled"])
    M = _log_uniform(rng, 1, 2048, 1)
    flops = 2 * M * K * N * {"gemm": 1, "mlp": 2, "gated": 3}[op]
    most = 40e9 if path == "actorder" else (150e9 if op == "gated" else 900e9)
    if flops > most:
        M = max(1, int(M * most / flops))
    graph = M <= 64 and op != "gemm"
    weights = K * N // 2 * {"gemm": 1, "mlp": 2, "gated": 3}[op]
    layers = max(1, min(8, int(240e6 / weights))) if graph else 1
    tp = rng.choice([1, 2, 4, 8]) if op != "gemm" else 1
    return _case(None, op, M, K, N, N2, G=G, tp=tp, dtype=dtype, path=path, layout=layout,
                 perm=op == "gemm" and path == "ordered" and rng.random() < 0.5, layers=layers, graph=graph)


# ---- inputs --------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _words(g, *shape):
    return torch.randint(-2**31, 2**31, shape, generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _layer(g, K, N, G, dtype, actorder, tp=1):
    """GPTQ-layout layer (qweight, scales, qzeros, g_idx): sorted rows, or K rows of a layer of tp * K rows
    in act-order (which keep the whole layer's groups)."""
    ng = -(-(K * (tp if actorder else 1)) // G)
    qw = _words(g, K // 8, N)
    sc = (torch.rand(ng, N, generator=g, device="cuda") * 0.018 + 0.002).to(dtype)
    qz = _words(g, ng, N // 8)
    if actorder:
        gi = (torch.randperm(K * tp, generator=g, device="cuda") // G)[:K].to(torch.int32).contiguous()
    else:
        gi = (torch.arange(K, device="cuda") // G).to(torch.int32)
    return qw, sc, qz, gi


def _x(g, M, K, dtype):
    return torch.randn(M, K, generator=g, device="cuda").to(dtype)


def _inputs(c, seed):
    """Each layer of the stack: (X, permutation or None, its weight matrices in GPTQ layout)."""
    g = _gen(seed)
    dt, act = DTYPES[c["dtype"]], c["path"] == "actorder"
    out = []
    for _ in range(c["layers"]):
        K, N, G = c["K"], c["N"], c["G"]
        P = None
        if not act and (c["op"] != "gemm" or c["perm"]):
            P = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
        ws = [_layer(g, K, N, G, dt, act)]
        if c["op"] == "gated":
            ws.append(_layer(g, K, N, G, dt, act))
            if act:  # gate and up read the same input: one act-order for both
                ws[1] = ws[1][:3] + (ws[0][3],)
        if c["op"] in ("mlp", "gated"):
            ws.append(_layer(g, N, c["N2"], G, dt, act, c["tp"]))
        out.append((_x(g, c["M"], K, dt), P, ws))
    return out


def _weight(c, layer):
    qw, sc, qz, gi = layer
    w = tpdq.QuantWeight.from_tensors(qw, sc, qz, gi, c["G"])
    return tpdq.pack_tiled(w) if c["layout"] == "tiled" else w


def _call(c, d):
    """One layer's call, as a program makes it with the buffers it keeps."""
    path = PATHS[c["path"]]
    if c["op"] == "gemm":
        return tpdq.w4a16_gemm(d["x"], d["w"][0], path, x_perm=d["p"], out=d["y"][0], workspace=d["ws"])
    fn = tpdq.mlp_shard if c["op"] == "mlp" else tpdq.gated_mlp_shard
    return fn(d["x"], *d["w"], path, P1=d["p"], y1=d["y"][0], y2=d["y"][1], workspace=d["ws"])


def prepare(case, seed):
    c = case
    if c["op"] == "reorder":
        g = _gen(seed)
        dt = DTYPES[c["dtype"]]
        w = [tpdq.QuantWeight.from_tensors(*_layer(g, k, n, c["G"], dt, True), c["G"])
             for k, n in ((c["K"], c["N"]), (c["N"], c["N2"]))]
        return {"case": c, "w": w, "ws": tpdq.Workspace(w[0].device)}
    dev = torch.device("cuda", torch.cuda.current_device())
    ws = tpdq.Workspace(dev)  # one scratch for the whole stack: its calls follow one another
    stack = []
    for x, p, layers in _inputs(c, seed):
        ys = [torch.zeros(c["M"], n, dtype=x.dtype, device=dev) for n in (c["N"], c["N2"]) if n]
        stack.append({"x": x, "p": p, "w": [_weight(c, l) for l in layers], "y": ys, "ws": ws})
    state = {"case": c, "stack": stack, "graph": None}
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):  # once outside the capture: kernels loaded, scratch grown
            for d in stack:
                _call(c, d)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for d in stack:
                _call(c, d)
        state["graph"] = graph
    return state


def run(state):
    c = state["case"]
    if c["op"] == "reorder":
        P1, g1, P2, g2, w1, w2 = tpdq.reorder(state["w"][0], state["w"][1], workspace=state["ws"])
        return {"P1": P1, "g1": g1, "P2": P2, "g2": g2, "qweight1": w1.qweight, "scales1": w1.scales,
                "qzeros1": w1.qzeros, "qweight2": w2.qweight}
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        for d in state["stack"]:
            _call(c, d)
    return [d["y"] for d in state["stack"]]


# ---- what a pass cannot do without, and what is right ----------------------

def work(case):
    c = case
    M, K, N, N2, G = c["M"], c["K"], c["N"], c["N2"], c["G"]
    act = c["path"] == "actorder"

    def layer(k, n, tp=1):
        ng = -(-(k * (tp if act else 1)) // G)
        return k * n // 2 + ng * n * 2 + ng * n // 2 + (4 * k if act else 0)

    if c["op"] == "reorder":
        ng1 = -(-K // G)
        w1 = K * N // 2 + ng1 * N * 2 + ng1 * N // 2
        return {"bytes": 2 * w1 + 2 * (N * N2 // 2) + 3 * 4 * (K + N), "flops": 0}
    perm = 4 * K if (c["perm"] or (c["op"] != "gemm" and not act)) else 0
    if c["op"] == "gemm":
        b, f = layer(K, N) + perm + 2 * M * (K + N), 2 * M * K * N
    else:
        first = 2 if c["op"] == "gated" else 1
        b = first * layer(K, N) + layer(N, N2, c["tp"]) + perm + 2 * M * (K + N + N2)
        f = 2 * M * (first * K * N + N * N2)
    return {"bytes": c["layers"] * b, "flops": c["layers"] * f}


def tolerance(case):
    """Whole numbers and copied bits are the same. fp16 and bf16 results: about four times the error of one
    rounding each of the weights, of Y1 and of Y2 to the type, which is what the library shows against 64 bits
    (fp16 2e-4 to 5e-4, bf16 2e-3 to 4e-3, the gated product the larger)."""
    if case["op"] == "reorder":
        return "exact"
    return {"rel": 1.6e-3 if case["dtype"] == "fp16" else 1.2e-2}


def _nibbles(w, dim):
    """int32 words -> the eight codes of each along `dim`."""
    s = torch.arange(0, 32, 4, device=w.device, dtype=torch.int32)
    shape = [1] * (w.dim() + 1)
    shape[dim + 1] = 8
    v = (w.unsqueeze(dim + 1) >> s.view(shape)) & 15
    return v.flatten(dim, dim + 1)


def _dequant(layer):
    qw, sc, qz, gi = layer
    g = gi.long()
    z = _nibbles(qz, 1).double()
    w = _nibbles(qw, 0).double()
    w -= z[g]
    w *= sc.double()[g]
    return w


def _pack(codes, dim):
    """Codes along `dim`, eight to a word, row 8r + j at bits 4j."""
    n = codes.shape[dim] // 8
    v = codes.unflatten(dim, (n, 8)).to(torch.int64)
    shape = [1] * v.dim()
    shape[dim + 1] = 8
    s = torch.arange(0, 32, 4, device=codes.device).view(shape)
    v = (v << s).sum(dim + 1)
    return torch.where(v >= 2**31, v - 2**32, v).to(torch.int32)


def exact(case, seed):
    c = case
    if c["op"] == "reorder":
        # integers and copied bits; P and the metadata in plain torch (the packed words' storage order is the
        # library's own)
        g = _gen(seed)
        dt = DTYPES[c["dtype"]]
        (q1, s1, z1, i1), (q2, s2, z2, i2) = [_layer(g, k, n, c["G"], dt, True)
                                              for k, n in ((c["K"], c["N"]), (c["N"], c["N2"]))]
        P1, P2 = torch.sort(i1, stable=True)[1], torch.sort(i2, stable=True)[1]
        zp = _pack(_nibbles(z1, 1)[:, P2], 1)
        return {"P1": P1.to(torch.int32), "g1": i1[P1], "P2": P2.to(torch.int32), "g2": i2[P2], "qweight1": None,
                "scales1": s1[:, P2].contiguous(), "qzeros1": zp, "qweight2": None}
    out = []
    for x, p, ws in _inputs(c, seed):
        xd = x.double()
        if p is not None:
            xd = xd[:, p.long()]
        y1 = xd @ _dequant(ws[0])
        if c["op"] == "gemm":
            out.append([y1])
            continue
        if c["op"] == "gated":
            y1 = torch.nn.functional.silu(y1) * (xd @ _dequant(ws[1]))
        out.append([y1, y1 @ _dequant(ws[-1])])
    return out
