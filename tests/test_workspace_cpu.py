"""What a call does with its workspace, from its recorded launches (no GPU):
every kernel stays inside the workspace and the outputs, and reads from the
workspace only what an earlier launch of the call left there."""
import os
import random

import pytest

from paper_2402_04925_amd import _abi
from tests import launches

if not os.path.exists(_abi.LIB_PATH):
    from paper_2402_04925_amd import build
    build.build()


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("recorder"))
    return lambda calls: launches.record(calls, d)


def _log_uniform(rng, lo, hi, step):
    return max(step, round(lo * (hi / lo) ** rng.random() / step) * step)


def _random_call(rng):
    op = rng.choice(["gemm", "gemm", "mlp", "gated", "noalloc"])
    step = rng.choice([8, 16, 128, 512])
    top = rng.choice([2000, 9000, 40000])
    K, N, N2 = (_log_uniform(rng, 8, top, step) for _ in range(3))
    G, path = rng.choice([8, 24, 32, 64, 128, 128, 256, 0]), rng.choice(["ordered", "ordered", "actorder", "global"])
    c = dict(op=op, M=_log_uniform(rng, 1, rng.choice([70, 300, 3000]), 1), K=K, N=N, N2=0 if op == "gemm" else N2,
             G=G, path=path, layout=rng.choice(["tiled", "gptq"]), dtype=rng.choice(["fp16", "bf16"]),
             perm=rng.random() < 0.4, gidx=path != "ordered" or G == 0 or rng.random() < 0.5)
    if rng.random() < 0.25:  # rows far apart: past 32-bit offsets from about 1000 rows on
        c["ldx"] = rng.choice([1 << 20, 1 << 21, 1 << 22])
    if G == 0:
        c["ng1"], c["ng2"] = rng.choice([5, 400]), rng.choice([5, 400])
    elif path != "ordered" and rng.random() < 0.5:  # a row shard of eight
        c["ng2"] = -(-N * 8 // G)
    return c


@pytest.mark.parametrize("ws", ["doc", 0, 4096, 1 << 20, 16 << 20, None])
def test_random_calls_stay_inside(record, ws):
    rng = random.Random(str(ws))
    calls = [dict(_random_call(rng), ws=ws) for _ in range(400)]
    done = 0
    for c, r in zip(calls, record(calls)):
        assert launches.outside(r) == [], c
        assert r["status"] in (_abi.OK, _abi.ERR_WORKSPACE, _abi.ERR_UNSUPPORTED), c
        assert ws != "doc" or c["op"] == "noalloc" or r["status"] != _abi.ERR_WORKSPACE, c
        done += r["status"] == _abi.OK
    assert done > 80


# Row-major X that the M-tiled kernel refuses (2 GiB or more) on large tiled
# weights is cut into launches of 64 rows; the last one, of 1 to 32 rows, takes
# the wide kernel, whose split-K partials the others do not use.
@pytest.mark.parametrize("op", ["mlp", "gated"])
@pytest.mark.parametrize("M", [131088, 131100])
def test_last_launch_of_many(record, op, M):
    (r,) = record([dict(op=op, M=M, K=8192, N=28672, N2=8192)])
    assert r["status"] == _abi.OK
    assert launches.outside(r) == []
    assert "k_wide" in r["launches"][-2]["kernel"] and "reduce" in r["launches"][-1]["kernel"]


@pytest.mark.parametrize("M,ldx", [(1040, 1 << 20), (1024, 1 << 20), (131082, 8192), (131072, 8192)])
@pytest.mark.parametrize("ws", [None, 4096])
def test_large_row_major_calls_need_their_workspace(record, M, ldx, ws):
    c = dict(op="gemm", M=M, K=8192, N=8192, ldx=ldx)
    short, full = record([dict(c, ws=ws), c])
    assert short["status"] == _abi.ERR_WORKSPACE and short["launches"] == []
    assert full["status"] == _abi.OK and launches.outside(full) == []


def test_route_does_not_depend_on_spare_workspace(record):
    """Any workspace of the documented size or more takes the same kernels with
    the same splits, so that results do not change with what other calls have
    made a shared workspace grow to."""
    rng = random.Random(7)
    calls = [dict(op="mlp", M=257, K=9224, N=2752, N2=40, G=24, path="actorder", layout="gptq", dtype="bf16"),
             dict(op="gemm", M=700, K=9224, N=2752, path="actorder", layout="gptq")]
    calls += [dict(c, M=rng.randint(1, 1500)) for c in (_random_call(rng) for _ in range(1500)) if c["op"] != "noalloc"]
    exact, spare = record(calls), record([dict(c, ws="2doc") for c in calls])
    much = record([dict(c, ws=4 << 30) for c in calls])
    for c, a, b, d in zip(calls, exact, spare, much):
        assert launches.route(a) == launches.route(b) == launches.route(d), c
    # ... and so does the library's own scratch, where the documented size fits
    mlp = [(c, r) for c, r in zip(calls, exact) if c["op"] == "mlp" and r["doc"] <= launches.SCRATCH_BYTES]
    for (c, r), n in zip(mlp, record([dict(c, op="noalloc") for c, _ in mlp])):
        assert launches.route(r) == launches.route(n), c


class _Library:
    """The library up to its launches: keeps the workspace bytes of each call."""

    def __init__(self, lib):
        self._lib, self.got = lib, []

    def __getattr__(self, name):
        if name in ("tpdq_w4a16_gemm", "tpdq_mlp_shard", "tpdq_gated_mlp_shard"):
            return lambda *args: self.got.append(args[-2]) or _abi.OK
        return getattr(self._lib, name)


def test_ordered_calls_ask_for_no_act_order_workspace(monkeypatch):
    """A layer of reorder() carries its sorted g_idx; an ordered call of it asks
    for what the same layer without one does, and an act-order call for more."""
    import torch
    import paper_2402_04925_amd as tpdq
    lib = _Library(_abi.lib())
    monkeypatch.setattr(_abi, "lib", lambda: lib)
    monkeypatch.setattr(tpdq, "_check_args", lambda *a, **k: None)
    monkeypatch.setattr(tpdq, "_stream_handle", lambda d: 0)

    def layer(K, N, gidx):
        G = 128
        return tpdq.QuantWeight(
            torch.empty(N // 16, tpdq.tiled_ld(K), dtype=torch.int32), torch.empty(K // G, N, dtype=torch.float16),
            torch.empty(K // G, N // 8, dtype=torch.int32),
            torch.zeros(K, dtype=torch.int32) if gidx else None, K, N, G, K // G, tpdq.LAYOUT_TILED)

    M, K, N = 300, 8192, 3584
    X, P = torch.empty(M, K, dtype=torch.float16), torch.zeros(K, dtype=torch.int32)

    def sizes(gidx, path):
        a, b = layer(K, N, gidx), layer(N, K, gidx)
        perm = P if path == tpdq.PATH_ORDERED else None
        lib.got.clear()
        tpdq.w4a16_gemm(X, a, path, x_perm=perm, workspace=tpdq.Workspace())
        tpdq.mlp_shard(X, a, b, path, P1=perm, workspace=tpdq.Workspace())
        tpdq.gated_mlp_shard(X, a, a, b, path, P1=perm, workspace=tpdq.Workspace())
        return list(lib.got)

    ordered = sizes(True, tpdq.PATH_ORDERED)
    assert len(ordered) == 3 and ordered == sizes(False, tpdq.PATH_ORDERED)
    assert all(a > o for a, o in zip(sizes(True, tpdq.PATH_ACTORDER), ordered))


@pytest.mark.parametrize("K,G", [(61440, 128), (65536, 128), (65536, 256), (81920, 256)])
@pytest.mark.parametrize("op,M", [("gemm", 1), ("gemm", 16), ("gemm", 64), ("gated", 4)])
def test_long_act_order_rows_keep_their_metadata_in_lds(record, K, G, op, M):
    """No act-order call whose tile's scales and zeros fit LDS reads them row by
    row from global memory (the third template argument)."""
    (r,) = record([dict(op=op, M=M, K=K, N=256, N2=0 if op == "gemm" else 512, G=G, path="actorder")])
    k = [l["kernel"] for l in r["launches"] if "k_rowmeta" in l["kernel"]][0]
    assert k.split(",")[2].strip() in ("2", "3"), k
    assert r["launches"][0]["lds"] <= 160 * 1024
