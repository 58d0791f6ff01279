"""The launches that a library call makes, without a GPU: libtpdq.so on the
stand-ins of launch_recorder.cpp, in a process of its own (in this one the
library may be bound to the real runtime already).

A call is a dict: op ("gemm", "mlp", "gated" or "noalloc"), M, K, N, N2, and
optionally G, path, layout, dtype, perm (gemm), gidx, ng1, ng2 (num_groups of
the first and second layer), ldx, and ws, its workspace: None for NULL, a
number of bytes, or "doc", "2doc" for (twice) what tpdq_workspace_bytes says.
"""
from __future__ import annotations

import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# far apart, so that what one tensor may hold never reaches the next
X_AT, WS_AT, Y1_AT, Y2_AT, W_AT = (i << 40 for i in range(1, 6))
SCRATCH_AT, SCRATCH_BYTES = 1 << 47, 64 << 20


def record(calls, tmpdir, root=ROOT):
    """[{status, doc, ws, launches}] of the calls."""
    so = os.path.join(tmpdir, "recorder.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-w",
                        "-I/opt/rocm/include", "-I" + os.path.join(root, "paper_2402_04925_amd", "csrc"),
                        os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-o", so], check=True)
    r = subprocess.run([sys.executable, "-c", "from tests import launches; launches._serve()"], cwd=ROOT,
                       input=json.dumps({"so": so, "root": root, "calls": calls}), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def outside(result):
    """The ranges that a call's launches write outside its workspace and
    outputs, or read from a workspace that no earlier launch has written."""
    bad, written = [], []
    ws, n = result["ws"]
    for l in result["launches"]:
        for kind, p, size in l["mem"]:
            in_ws = ws <= p and p + size <= ws + n
            if kind == "unknown":
                bad.append((l["kernel"], kind))
            elif kind == "w":
                if not in_ws and not any(a <= p and p + size <= a + b for a, b in result["out"]):
                    bad.append((l["kernel"], "write", p - ws, size, n))
                if in_ws:
                    written = [(a, b, k) for a, b, k in written if b <= p or p + size <= a]
                    written.append((p, p + size, l["kernel"]))
            elif in_ws and not any(a <= p and p + size <= b for a, b, _ in written):
                bad.append((l["kernel"], "read of what no launch left there", p - ws, size))
    return bad


def route(result):
    return [(l["kernel"], l["grid"], l["block"]) for l in result["launches"]]


def _layer(abi, K, N, c, ng, at):
    G = c.get("G", 128)
    tiled = c.get("layout", "tiled") == "tiled"
    return abi.W4(qweight=at, ld_q=(K + 127) // 128 * 256 if tiled else N, scales=at + (1 << 36), ld_s=N,
                  qzeros=at + (2 << 36), ld_z=N // 8, g_idx=at + (3 << 36) if c.get("gidx", True) else None,
                  K=K, N=N, group_size=G, num_groups=ng or -(-K // max(G, 8)),
                  layout=abi.LAYOUT_TILED if tiled else abi.LAYOUT_GPTQ, zero_offset=0)


def _call(abi, lib, c):
    M, K, N, N2 = c["M"], c["K"], c["N"], c.get("N2", 0)
    path = {"ordered": abi.PATH_ORDERED, "actorder": abi.PATH_ACTORDER,
            "global": abi.PATH_ACTORDER_GLOBAL}[c.get("path", "ordered")]
    dt = abi.BF16 if c.get("dtype", "fp16") == "bf16" else abi.FP16
    op = c["op"]
    w1, w2 = _layer(abi, K, N, c, c.get("ng1"), W_AT), _layer(abi, N, N2, c, c.get("ng2"), W_AT + (4 << 36))
    up = _layer(abi, K, N, c, c.get("ng1"), W_AT + (8 << 36))
    b = ctypes.byref
    code = {"gemm": abi.OP_GEMM, "gated": abi.OP_GATED_MLP}.get(op, abi.OP_MLP)
    doc = lib.tpdq_workspace_bytes(code, M, b(w1), None if op == "gemm" else b(w2))
    ws = c.get("ws", "doc")
    n = 0 if ws is None else {"doc": doc, "2doc": 2 * doc}.get(ws, ws)
    at = None if ws is None else WS_AT
    ldx = c.get("ldx", K)
    if op == "gemm":
        st = lib.tpdq_w4a16_gemm(X_AT, ldx, M, W_AT + (12 << 36) if c.get("perm") else None, b(w1), path, dt,
                                 Y1_AT, N, at, n, None)
    else:
        P1 = W_AT + (12 << 36) if path == abi.PATH_ORDERED else None
        if op == "mlp":
            st = lib.tpdq_mlp_shard(X_AT, ldx, M, P1, b(w1), b(w2), path, dt, Y1_AT, Y2_AT, at, n, None)
        elif op == "gated":
            st = lib.tpdq_gated_mlp_shard(X_AT, ldx, M, P1, b(w1), b(up), b(w2), path, dt, Y1_AT, Y2_AT, at, n,
                                          None)
        else:
            st = lib.tpdq_mlp_shard_noalloc(X_AT, ldx, M, P1, b(w1), b(w2), path, dt, Y1_AT, Y2_AT, None)
            at, n = SCRATCH_AT, SCRATCH_BYTES
    return {"status": st, "doc": doc, "ws": [at or 0, n], "out": [[Y1_AT, 2 * M * N], [Y2_AT, 2 * M * N2]],
            "launches": json.loads(lib._recorder.recorder_take().decode())}


def _serve():
    req = json.load(sys.stdin)
    sys.path.insert(0, req["root"])
    rec = ctypes.CDLL(req["so"], mode=ctypes.RTLD_GLOBAL)
    rec.recorder_take.restype = ctypes.c_char_p
    from paper_2402_04925_amd import _abi
    lib = _abi._declare(ctypes.CDLL(os.path.join(req["root"], "paper_2402_04925_amd", "libtpdq.so")))
    lib._recorder = rec
    print(json.dumps([_call(_abi, lib, c) for c in req["calls"]]))
