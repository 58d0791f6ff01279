"""Per-row metadata where LDS holds the tile's scales and zeros but not every
row's group too (long K, or more than 1024 groups): the groups come from
g_idx, or from k / G where sorted rows have none."""
import numpy as np
import pytest

from oracle import tpdq_oracle as o
from paper_2402_04925_amd import inputs
from tests.gpu_util import layer_to_dev, log, np_of, to_dev, torch_dev

pytestmark = pytest.mark.gpu

# max|err| / max|ref|: weights rounded once (2^-12, 2^-9 relative; a random
# walk over K) and the result once
TOL = {"fp16": 2.0**-10, "bf16": 2.0**-7}


def _layer(K, N, G, dtype, seed):
    sd = np.float16 if dtype == "fp16" else inputs.BF16
    return inputs.make_layer(K, N, G, 100, 0, 20, 30, 40, seed=seed, scale_dtype=sd)


def _x(M, K, dtype):
    return inputs.random_activations(M, K, np.random.default_rng(M + K),
                                     np.float16 if dtype == "fp16" else inputs.BF16)


def _deq(l):
    return o.dequant(l.qweight, l.scales, l.qzeros, l.g_idx)


# one row past 1024 groups, a long K; one to four row tiles, X as it is and in
# operand order (from 17 rows); columns short of and past a tile
@pytest.mark.parametrize("K,N,G", [(8200, 24, 8), (65664, 40, 128)])
@pytest.mark.parametrize("M", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("layout,dtype", [("gptq", "fp16"), ("tiled", "fp16"), ("gptq", "bf16"), ("tiled", "bf16")])
def test_actorder(K, N, G, M, layout, dtype):
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"rowmeta idx K={K} N={N} G={G} M={M} {layout} {dtype}")
    l = _layer(K, N, G, dtype, K)
    w = layer_to_dev(l, dev)
    if layout == "tiled":
        w = tpdq.pack_tiled(w)
    X = _x(M, K, dtype)
    y = tpdq.w4a16_gemm(to_dev(X, dev, dtype == "bf16"), w, tpdq.PATH_ACTORDER)
    torch.cuda.synchronize()
    assert o.rel_err(np_of(y), X.astype(np.float64) @ _deq(l)) <= TOL[dtype]


@pytest.mark.parametrize("M", [2, 20, 40])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_gated_row_shards(M, dtype):
    """Gate and up with more than 1024 groups of few rows (what a row shard
    keeps), and sorted rows in groups of 8 without a g_idx."""
    import torch
    import paper_2402_04925_amd as tpdq
    dev = torch_dev()
    log(f"rowmeta idx gated M={M} {dtype}")
    tp, K, N = 8, 1032, 136
    whole = [_layer(tp * K, N, 8, dtype, s) for s in (1, 2)]
    whole[1].g_idx = whole[0].g_idx
    down = _layer(N, 64, 8, dtype, 3)
    ws = [layer_to_dev(l, dev).row_shard(1, tp, False) for l in whole] + [layer_to_dev(down, dev)]
    assert ws[0].num_groups > 1024
    X = _x(M, K, dtype)
    Xd = to_dev(X, dev, dtype == "bf16")
    y1, _ = tpdq.gated_mlp_shard(Xd, *ws, tpdq.PATH_ACTORDER)
    x = X.astype(np.float64)
    wg, wu = (_deq(l)[K:2 * K] for l in whole)
    assert o.rel_err(np_of(y1), o.silu(x @ wg) * (x @ wu)) <= TOL[dtype]

    Ks = 8264
    s = _layer(Ks, 24, 8, dtype, 4)
    s.g_idx = (np.arange(Ks) // 8).astype(np.int32)
    Xs = _x(M, Ks, dtype)
    y = tpdq.w4a16_gemm(to_dev(Xs, dev, dtype == "bf16"), layer_to_dev(s, dev, with_gidx=False), tpdq.PATH_ORDERED)
    torch.cuda.synchronize()
    assert o.rel_err(np_of(y), Xs.astype(np.float64) @ _deq(s)) <= TOL[dtype]
