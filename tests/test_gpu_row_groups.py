"""Row groups of the ordered decode kernel (17 to 256 rows in one launch): every
split of row and column tiles, both layouts, X as it is, gathered, or copied to
operand order, with and without a workspace, and the MLP whose GEMM1 writes
Y1 in GEMM2's operand order."""
import ctypes

import numpy as np
import pytest

from oracle import tpdq_oracle as o
from paper_2402_04925_amd import inputs
from tests.gpu_util import layer_to_dev, log, np_of, to_dev, torch_dev

pytestmark = pytest.mark.gpu

# max|err| / max|ref|: the result's rounding (2^-12, 2^-9), doubled for fp32
# sums in another order near a rounding boundary; an MLP's Y1 is rounded too
TOL = {"fp16": 2.0**-10, "bf16": 2.0**-7}


def _sorted(K, N, G, dtype, seed):
    l = inputs.make_layer(K, N, G, 100, 0, 20, 30, 40, seed=seed,
                          scale_dtype=np.float16 if dtype == "fp16" else inputs.BF16)
    l.g_idx = (np.arange(K) // G).astype(np.int32)
    return l


def _x(M, K, dtype):
    return inputs.random_activations(M, K, np.random.default_rng(M + K),
                                     np.float16 if dtype == "fp16" else inputs.BF16)


def _deq(l):
    return o.dequant(l.qweight, l.scales, l.qzeros, l.g_idx)


# column tiles short of, at and past the widths of 1 to 4 tiles per workgroup
# (N = 8 half a tile; 2056 past 128 tiles; 3464 and 8200 the wider ones); K
# shorter than the waves' runs, ragged, and with a partial last group
@pytest.mark.parametrize("K,N,G", [(256, 8, 32), (1000, 264, 128), (264, 2056, 64), (512, 3464, 128), (384, 8200, 256)])
@pytest.mark.parametrize("M", [17, 32, 33, 64, 65, 129, 256, 257])
@pytest.mark.parametrize("layout,dtype", [("tiled", "fp16"), ("gptq", "fp16"), ("tiled", "bf16"), ("gptq", "bf16")])
def test_row_groups(K, N, G, M, layout, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    from paper_2402_04925_amd import _abi
    dev = torch_dev()
    log(f"row groups K={K} N={N} G={G} M={M} {layout} {dtype}")
    l = _sorted(K, N, G, dtype, K + N)
    w = layer_to_dev(l, dev, with_gidx=False)
    if layout == "tiled":
        w = tpdq.pack_tiled(w)
    X = _x(M, K, dtype)
    Xd = to_dev(X, dev, dtype == "bf16")
    perm = np.random.default_rng(1).permutation(K).astype(np.int32)
    y = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED)
    yp = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED, x_perm=to_dev(perm, dev))
    yn = torch.empty_like(y)
    c = w.c_struct()
    _abi.check(_abi.lib().tpdq_w4a16_gemm(
        Xd.data_ptr(), K, M, None, ctypes.byref(c), tpdq.PATH_ORDERED, tpdq.FP16 if dtype == "fp16" else tpdq.BF16,
        yn.data_ptr(), N, None, 0, torch.cuda.current_stream(dev).cuda_stream))
    torch.cuda.synchronize()
    W = _deq(l)
    x = X.astype(np.float64)
    tol = TOL[dtype] if M < 256 else 2 * TOL[dtype]  # tiled prefill sizes round the weights
    assert o.rel_err(np_of(y), x @ W) <= tol
    assert o.rel_err(np_of(yn), x @ W) <= tol
    assert o.rel_err(np_of(yp), x[:, perm] @ W) <= tol


@pytest.mark.parametrize("M", [33, 100, 256])
@pytest.mark.parametrize("layout", ["tiled", "gptq"])
@pytest.mark.parametrize("gated", [False, True])
def test_mlp_row_groups(M, layout, gated):
    """Y1 goes through the workspace in operand order where N1 % 128 == 0."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    for N1 in (1152, 1160):
        K1, N2 = 520, 264
        first = [_sorted(K1, N1, 64, "fp16", 1 + i) for i in range(2 if gated else 1)]
        down = _sorted(N1, N2, 32, "fp16", 9)
        X = _x(M, K1, "fp16")
        P1 = np.random.default_rng(2).permutation(K1).astype(np.int32)
        ws = [layer_to_dev(l, dev, with_gidx=False) for l in first + [down]]
        if layout == "tiled":
            ws = [tpdq.pack_tiled(w) for w in ws]
        call = tpdq.gated_mlp_shard if gated else tpdq.mlp_shard
        y1, y2 = call(to_dev(X, dev), *ws, tpdq.PATH_ORDERED, P1=to_dev(P1, dev))
        torch.cuda.synchronize()
        x = X[:, P1].astype(np.float64)
        e1 = x @ _deq(first[0])
        if gated:
            e1 = o.silu(e1) * (x @ _deq(first[1]))
        assert o.rel_err(np_of(y1), e1) <= 2 * TOL["fp16"], N1
        # Y2 of the Y1 that the call rounded
        assert o.rel_err(np_of(y2), np_of(y1).astype(np.float64) @ _deq(down)) <= 2 * TOL["fp16"], N1


# 38 (49) blocks of 128 rows, 9 to 13 to a wave, the last one ragged: whole chunks
# of four, the reload of the metadata and a ragged last chunk; from 33 rows on X
# without a perm is copied to operand order. tests/test_plans_cpu.py has the
# kernels that these calls reach.
LONG = [(K, N, G, M, layout, dtype) for K, N, G, M in
        [(4744, 12296, G, M) for G in (32, 64, 128, 256) for M in (17, 64, 100, 250)] + [(6200, 4104, 128, 33)]
        for dtype in ("fp16", "bf16") for layout in ("tiled", "gptq")]
_long = {}


@pytest.mark.parametrize("K,N,G,M,layout,dtype", LONG)
def test_long_rows(K, N, G, M, layout, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"long rows K={K} N={N} G={G} M={M} {layout} {dtype}")
    if _long.get("key") != (K, N, G, dtype):
        l = _sorted(K, N, G, dtype, G)
        # whole octets of columns: the first and last tiles and 12 others
        octets = np.unique(np.concatenate([[0, 1, N // 8 - 2, N // 8 - 1],
                                           np.random.default_rng(G).integers(0, N // 8, 12)]))
        cols = (8 * octets[:, None] + np.arange(8)).ravel()
        W = o.dequant(np.ascontiguousarray(l.qweight[:, cols]), np.ascontiguousarray(l.scales[:, cols]),
                      np.ascontiguousarray(l.qzeros[:, octets]), l.g_idx)
        w = layer_to_dev(l, dev, with_gidx=False)
        _long.update(key=(K, N, G, dtype), cols=cols, W=W, w={"gptq": w, "tiled": tpdq.pack_tiled(w)})
    w, cols, W = _long["w"][layout], _long["cols"], _long["W"]
    X = _x(M, K, dtype)
    Xd = to_dev(X, dev, dtype == "bf16")
    perm = np.random.default_rng(1).permutation(K).astype(np.int32)
    x = X.astype(np.float64)
    y = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED)
    assert o.rel_err(np_of(y)[:, cols], x @ W) <= TOL[dtype]
    assert torch.equal(y, tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED))
    yp = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED, x_perm=to_dev(perm, dev))
    assert o.rel_err(np_of(yp)[:, cols], x[:, perm] @ W) <= TOL[dtype]
    if layout == "gptq":  # X as it is: no workspace for a copy
        yn = torch.empty_like(y)
        c = w.c_struct(tpdq.PATH_ORDERED)
        from paper_2402_04925_amd import _abi
        _abi.check(_abi.lib().tpdq_w4a16_gemm(
            Xd.data_ptr(), K, M, None, ctypes.byref(c), tpdq.PATH_ORDERED,
            tpdq.FP16 if dtype == "fp16" else tpdq.BF16, yn.data_ptr(), N, None, 0,
            torch.cuda.current_stream(dev).cuda_stream))
        assert o.rel_err(np_of(yn)[:, cols], x @ W) <= TOL[dtype]
