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
