"""Per-row metadata at more than 64 rows (dequantized once to 16 bits, then a
dense MFMA GEMM): act-order and sorted rows in groups that are not whole
32-row steps, column chunks, K splits, the gated product, and the decode
route of a call whose workspace is too small for it."""
import ctypes

import numpy as np
import pytest

from oracle import tpdq_oracle as o
from paper_2402_04925_amd import inputs
from tests.gpu_util import layer_to_dev, log, np_of, to_dev, torch_dev

pytestmark = pytest.mark.gpu

# max|err| / max|ref|: weights rounded once (2^-12, 2^-9 relative; a random
# walk over K) and the result once (2^-12, 2^-9)
TOL = {"fp16": 2.0**-10, "bf16": 2.0**-7}


def _layer(K, N, G, dtype, seed):
    sd = np.float16 if dtype == "fp16" else inputs.BF16
    return inputs.make_layer(K, N, G, 100, 0, 20, 30, 40, seed=seed, scale_dtype=sd)


def _x(M, K, dtype):
    return inputs.random_activations(M, K, np.random.default_rng(M + K),
                                     np.float16 if dtype == "fp16" else inputs.BF16)


def _deq(l):
    return o.dequant(l.qweight, l.scales, l.qzeros, l.g_idx)


def _gemm(tpdq, X, w, path, nbytes, perm=None):
    """w4a16_gemm with a workspace of nbytes exactly."""
    import torch
    from paper_2402_04925_amd import _abi
    y = torch.empty(X.shape[0], w.N, dtype=X.dtype, device=X.device)
    buf = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=X.device)
    c = w.c_struct()
    _abi.check(_abi.lib().tpdq_w4a16_gemm(
        X.data_ptr(), X.stride(0), X.shape[0], None if perm is None else perm.data_ptr(), ctypes.byref(c),
        path, tpdq.FP16 if X.dtype == torch.float16 else tpdq.BF16, y.data_ptr(), w.N, buf.data_ptr(), nbytes,
        torch.cuda.current_stream(X.device).cuda_stream))
    torch.cuda.synchronize()
    return y


# one row past the decode kernels (which small layers take up to 256 rows:
# tests/test_plans_cpu.py) and past those, ragged rows and columns (N % 16 == 8, a
# 512-column tile plus 8), a ragged last block of K, groups of 8 and as many
# of them as don't fit in LDS, 128-row tiles
@pytest.mark.parametrize("K,N,G,M", [
    (256, 24, 32, 65), (1000, 520, 128, 130), (1064, 1032, 8, 129), (3072, 72, 8, 70), (4096, 512, 64, 260),
    (512, 2568, 128, 1100), (256, 24, 32, 257), (3072, 72, 8, 300),
])
@pytest.mark.parametrize("layout", ["gptq", "tiled"])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_actorder(K, N, G, M, layout, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"dense16 K={K} N={N} G={G} M={M} {layout} {dtype}")
    l = _layer(K, N, G, dtype, K + N)
    X = _x(M, K, dtype)
    w = layer_to_dev(l, dev)
    if layout == "tiled":
        w = tpdq.pack_tiled(w)
    Xd = to_dev(X, dev, dtype == "bf16")
    y = [tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ACTORDER) for _ in range(2)]
    perm = np.random.default_rng(3).permutation(K).astype(np.int32)
    yp = tpdq.w4a16_gemm(Xd, w, tpdq.PATH_ACTORDER, x_perm=to_dev(perm, dev))
    torch.cuda.synchronize()
    W = _deq(l)
    assert torch.equal(y[0], y[1])
    assert o.rel_err(np_of(y[0]), X.astype(np.float64) @ W) <= TOL[dtype]
    assert o.rel_err(np_of(yp), X[:, perm].astype(np.float64) @ W) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("M", [100, 300])
def test_column_chunks_and_small_workspaces(dtype, M):
    """Three chunks of 512 columns (the last of 136), and the decode kernels
    where not even one fits: the same weights, so the same result up to the
    order of the fp32 sums."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    K, N, G = 1032, 1160, 64
    l = _layer(K, N, G, dtype, 9)
    X = _x(M, K, dtype)
    w, Xd = layer_to_dev(l, dev), to_dev(X, dev, dtype == "bf16")
    ref = X.astype(np.float64) @ _deq(l)
    chunk = 9 * 256 * 512
    for nbytes in (chunk + 4096, chunk, chunk - 256, 0):
        y = _gemm(tpdq, Xd, w, tpdq.PATH_ACTORDER, nbytes)
        assert o.rel_err(np_of(y), ref) <= TOL[dtype], nbytes


@pytest.mark.parametrize("G", [0, 24, 8])
@pytest.mark.parametrize("M", [77, 270])
def test_sorted_rows_of_other_groups(G, M):
    """The ordered path where groups are not whole 32-row steps."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    K, N = 1008, 136
    l = inputs.make_unequal_layer(K, N, 11, seed=4) if G == 0 else _layer(K, N, G, "fp16", G)
    P, gs, _, _, wo, _ = tpdq.reorder(layer_to_dev(l, dev), layout=tpdq.LAYOUT_TILED)
    X = _x(M, K, "fp16")
    y = tpdq.w4a16_gemm(to_dev(X, dev), wo, tpdq.PATH_ORDERED, x_perm=P)
    torch.cuda.synchronize()
    assert o.rel_err(np_of(y), X.astype(np.float64) @ _deq(l)) <= TOL["fp16"]


@pytest.mark.parametrize("M,K,N", [(66, 264, 264), (300, 4096, 520), (259, 264, 264)])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_gated_actorder(M, K, N, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"dense16 gated M={M} K={K} N={N} {dtype}")
    gate, up, down = _layer(K, N, 64, dtype, 1), _layer(K, N, 64, dtype, 2), _layer(N, 64, 8, dtype, 3)
    up.g_idx = gate.g_idx
    X = _x(M, K, dtype)
    y1, _ = tpdq.gated_mlp_shard(to_dev(X, dev, dtype == "bf16"),
                                 *(layer_to_dev(l, dev) for l in (gate, up, down)), tpdq.PATH_ACTORDER)
    torch.cuda.synchronize()
    x = X.astype(np.float64)
    assert o.rel_err(np_of(y1), o.silu(x @ _deq(gate)) * (x @ _deq(up))) <= TOL[dtype]
