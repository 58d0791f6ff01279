"""The M-tiled GEMM with exact weights (the gated product, and smaller weights
below prefill sizes; M > 64), its K splits, and the routes by workspace."""
import ctypes

import numpy as np
import pytest

from oracle import tpdq_oracle as o
from paper_2402_04925_amd import inputs
from tests.gpu_util import layer_to_dev, log, np_of, to_dev, torch_dev

pytestmark = pytest.mark.gpu

# max|err| / max|ref|: one rounding of the result to the type (2^-11, 2^-8
# halved), twice that for fp32 sums in another order near a rounding boundary
TOL = {"fp16": 2.0**-10, "bf16": 2.0**-7}

# K, N, G, M: the smallest M, whole and ragged tiles of rows and columns (N
# past a 512- and a 256-column tile by 8), a ragged last block of K and a
# partial last group, every group size (G = 256 spans two blocks, cut by the K
# split at an odd block), K too short to split
SHAPES = [
    (1024, 520, 128, 65), (1000, 264, 32, 128), (1064, 1032, 64, 129), (2432, 136, 256, 255),
    (128, 512, 128, 77), (4096, 8, 128, 66),
]


def _layers(K, N, G, dtype, n):
    sd = np.float16 if dtype == "fp16" else inputs.BF16
    ls = [inputs.make_layer(K, N, G, 100, 0, 20 + i, 30 + i, 40 + i, seed=K + N + G, scale_dtype=sd)
          for i in range(n)]
    for l in ls:
        l.g_idx = (np.arange(K) // G).astype(np.int32)   # sorted rows
    return ls


def _x(M, K, dtype):
    return inputs.random_activations(M, K, np.random.default_rng(M + K),
                                     np.float16 if dtype == "fp16" else inputs.BF16)


def _product(X, l):
    return X.astype(np.float64) @ o.dequant(l.qweight, l.scales, l.qzeros, l.g_idx)


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("K,N,G,M", SHAPES)
def test_exact_gemm(K, N, G, M, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"exact M-tiled K={K} N={N} G={G} M={M} {dtype}")
    (l,) = _layers(K, N, G, dtype, 1)
    X = _x(M, K, dtype)
    w = tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False))
    perm = np.random.default_rng(5).permutation(K).astype(np.int32)
    Xd = to_dev(X, dev, dtype == "bf16")
    y = [tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED) for _ in range(2)]
    yp = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED, x_perm=to_dev(perm, dev))
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1])
    assert o.rel_err(np_of(y[0]), _product(X, l)) <= TOL[dtype]
    assert o.rel_err(np_of(yp), _product(X[:, perm], l)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("K,N,G,M", SHAPES)
def test_exact_gated(K, N, G, M, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"exact M-tiled gated K={K} N={N} G={G} M={M} {dtype}")
    gate, up = _layers(K, N, G, dtype, 2)
    down = _layers(N, 64, 8, dtype, 1)[0]
    X = _x(M, K, dtype)
    ws = [tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False)) for l in (gate, up, down)]
    P1 = np.random.default_rng(6).permutation(K).astype(np.int32)
    y1, _ = tpdq.gated_mlp_shard(to_dev(X, dev, dtype == "bf16"), *ws, tpdq.PATH_ORDERED,
                                 P1=to_dev(P1, dev))
    torch.cuda.synchronize()
    ref = o.silu(_product(X[:, P1], gate)) * _product(X[:, P1], up)
    assert o.rel_err(np_of(y1), ref) <= TOL[dtype]


# M >= 256: 64-row tiles and K splits where 128-row tiles leave CUs idle; 128
# rows with a split; the unsplit 128-row tiles of a call without a workspace
@pytest.mark.parametrize("M,K,N", [(256, 1024, 1024), (300, 4096, 1032), (1030, 2048, 4096), (700, 8192, 520)])
@pytest.mark.parametrize("workspace", [True, False])
def test_prefill_splits_and_null_workspace(M, K, N, workspace):
    import torch
    import paper_2402_04925_amd as tpdq
    from paper_2402_04925_amd import _abi
    dev = torch_dev()
    log(f"prefill splits M={M} K={K} N={N} workspace={workspace}")
    (l,) = _layers(K, N, 128, "fp16", 1)
    X = _x(M, K, "fp16")
    w = tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False))
    Xd = to_dev(X, dev)
    if workspace:
        y = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ORDERED)
    else:
        y = torch.empty(M, N, dtype=torch.float16, device=dev)
        c = w.c_struct()
        _abi.check(_abi.lib().tpdq_w4a16_gemm(
            Xd.data_ptr(), K, M, None, ctypes.byref(c), tpdq.PATH_ORDERED, tpdq.FP16, y.data_ptr(), N,
            None, 0, torch.cuda.current_stream(dev).cuda_stream))
    torch.cuda.synchronize()
    # weights rounded to fp16 (2^-11 each, a random walk over K) and the result once
    assert o.rel_err(np_of(y), _product(X, l)) <= 2.0**-9


@pytest.mark.parametrize("M", [65, 200])
def test_small_workspace_keeps_its_route(M):
    """The base route's workspace is still accepted and gives the same result
    up to one rounding (no perm: none at all)."""
    import torch
    import paper_2402_04925_amd as tpdq
    from paper_2402_04925_amd import _abi
    dev = torch_dev()
    K, N = 1024, 264
    (l,) = _layers(K, N, 128, "fp16", 1)
    X = _x(M, K, "fp16")
    w = tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False))
    Xd = to_dev(X, dev)
    y = torch.empty(M, N, dtype=torch.float16, device=dev)
    c = w.c_struct()
    lib = _abi.lib()
    _abi.check(lib.tpdq_w4a16_gemm(Xd.data_ptr(), K, M, None, ctypes.byref(c), tpdq.PATH_ORDERED, tpdq.FP16,
                                   y.data_ptr(), N, None, 0, torch.cuda.current_stream(dev).cuda_stream))
    P = torch.randperm(K, device=dev).to(torch.int32)
    yp = torch.empty_like(y)
    nbytes = 4 * ((K + 127) // 128) * 4096   # the decode route's gather of 64 rows
    buf = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    assert nbytes < lib.tpdq_workspace_bytes(_abi.OP_GEMM, M,
                                             ctypes.byref(c), None)
    _abi.check(lib.tpdq_w4a16_gemm(Xd.data_ptr(), K, M, P.data_ptr(), ctypes.byref(c), tpdq.PATH_ORDERED,
                                   tpdq.FP16, yp.data_ptr(), N, buf.data_ptr(), nbytes,
                                   torch.cuda.current_stream(dev).cuda_stream))
    torch.cuda.synchronize()
    assert o.rel_err(np_of(y), _product(X, l)) <= TOL["fp16"]
    assert o.rel_err(np_of(yp), _product(X[:, np_of(P)], l)) <= TOL["fp16"]


# 64-row tiles at prefill sizes, without and with a K split, whole and ragged,
# every group size; 64-row tiles of large weights below them
NOT_FINITE = [(300, 4096, 1032, 128), (256, 1000, 264, 32), (700, 8192, 520, 256), (257, 1064, 1160, 64),
              (300, 512, 8192, 128), (64, 8192, 8200, 128)]


@pytest.mark.parametrize("M,K,N,G", NOT_FINITE)
def test_not_finite_activations(M, K, N, G):
    """bf16: an infinite x gives each column +-Inf (NaN where the weight is 0),
    a very large one its finite product, and the other rows are as without."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"not finite M={M} K={K} N={N} G={G}")
    (l,) = _layers(K, N, G, "bf16", 1)
    w = tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False))
    X = _x(M, K, "bf16")
    clean = tpdq.w4a16_gemm(to_dev(X, dev, True), w, tpdq.PATH_ORDERED)
    X[3, 5], X[M - 1, K - 1] = np.inf, -np.inf
    X[17, 33], X[17, K - 2] = 2.0**126, -(2.0**125)
    bad = [3, 17, M - 1]
    y = tpdq.w4a16_gemm(to_dev(X, dev, True), w, tpdq.PATH_ORDERED)
    torch.cuda.synchronize()
    rest = [m for m in range(M) if m not in bad]
    assert torch.equal(y[rest], clean[rest])
    W = o.dequant(l.qweight, l.scales, l.qzeros, l.g_idx)
    with np.errstate(invalid="ignore"):
        ref = X[bad].astype(np.float64) @ W
    got = np_of(y[bad])
    for i in (0, 2):
        np.testing.assert_array_equal(got[i], ref[i])
    # weights rounded to bf16 (2^-9 each) and the result once
    assert np.isfinite(got[1]).all() and o.rel_err(got[1], ref[1]) <= 2.0**-7


def test_not_finite_activations_gated():
    """The gate overflows its sums, the up projection scales it back."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    M, K, N = 130, 1064, 520
    gate, up = _layers(K, N, 128, "bf16", 2)
    up.scales = (up.scales * 2.0**-120).astype(up.scales.dtype)
    down = _layers(N, 64, 8, "bf16", 1)[0]
    X = _x(M, K, "bf16")
    X[7, 9] = 2.0**124
    ws = [tpdq.pack_tiled(layer_to_dev(l, dev, with_gidx=False)) for l in (gate, up, down)]
    y1, _ = tpdq.gated_mlp_shard(to_dev(X, dev, True), *ws, tpdq.PATH_ORDERED,
                                 P1=to_dev(np.arange(K, dtype=np.int32), dev))
    torch.cuda.synchronize()
    with np.errstate(over="ignore"):
        ref = o.silu(_product(X[7:8], gate)) * _product(X[7:8], up)
    got = np_of(y1[7:8])
    # both products of bf16 weights (2^-9 each), one rounding
    assert np.isfinite(got).all() and o.rel_err(got, ref) <= 2.0**-6
