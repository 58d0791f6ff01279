"""Which kernels calls of a size take, from their recorded launches (no GPU)."""
import os

import pytest

from paper_2402_04925_amd import _abi
from tests import launches
from tests.test_gpu_row_groups import LONG

if not os.path.exists(_abi.LIB_PATH):
    from paper_2402_04925_amd import build
    build.build()


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("recorder"))
    return lambda calls: launches.record(calls, d)


def _ordered(result):
    """(row tiles, column tiles, prepared X, grid) of a call's ordered launches."""
    out = []
    for l in result["launches"]:
        if l["kernel"].startswith("k_ordered"):
            a = l["kernel"].split("<")[1].split(",")
            out.append((int(a[0]), int(a[5]), a[3].strip() == "3", l["grid"]))
    return out


def test_long_rows_reach_what_they_test(record):
    """The calls of test_gpu_row_groups.test_long_rows: one, two and four row
    tiles in both layouts, from the copy in operand order and from X as it is."""
    calls = [dict(op="gemm", M=M, K=K, N=N, G=G, layout=layout, dtype=dtype, gidx=False,
                  perm=perm, ws="doc") for K, N, G, M, layout, dtype in LONG for perm in (False, True)]
    seen = {"tiled": set(), "gptq": set()}
    for c, r in zip(calls, record(calls)):
        seen[c["layout"]] |= {(mt, prep) for mt, _, prep, _ in _ordered(r)}
    for layout in seen:
        assert {mt for mt, _ in seen[layout]} == {1, 2, 4}, layout
        assert {prep for _, prep in seen[layout]} == {True, False}, layout


# Row groups of one tile read GPTQ-layout weights of G = 32 once per 16 rows:
# 5248 x 20608 at M = 1000 took 1841 us where launches of 64 rows with all four
# row tiles had taken 1245
@pytest.mark.parametrize("K,N,M", [(5248, 20608, 1000), (1024, 24064, 128), (2560, 30208, 48), (8192, 8192, 1500)])
@pytest.mark.parametrize("G,dtype", [(32, "fp16"), (32, "bf16"), (256, "fp16")])
def test_many_rows_share_their_weights(record, K, N, M, G, dtype):
    (r,) = record([dict(op="gemm", M=M, K=K, N=N, G=G, layout="gptq", dtype=dtype, gidx=False, perm=True)])
    for mt, tn, _, grid in _ordered(r):
        assert mt >= 2


# Two row and four column tiles take the registers of a whole CU: on grids of
# many rounds no second workgroup covers its waits (2304 x 26368 at M = 100, 38.7
# -> 54.5 us)
@pytest.mark.parametrize("K,N,M", [(2304, 26368, 33), (2176, 25216, 64), (512, 14848, 64)])
@pytest.mark.parametrize("layout,G", [("tiled", 128), ("tiled", 256), ("gptq", 256)])
def test_many_rounds_take_two_workgroups_per_cu(record, K, N, M, layout, G):
    (r,) = record([dict(op="gemm", M=M, K=K, N=N, G=G, layout=layout, gidx=False, perm=True)])
    assert all((mt, tn) != (2, 4) or grid <= 256 for mt, tn, _, grid in _ordered(r))


# 17 to 64 rows on few columns: row groups over the whole K left most CUs idle
# (65536 x 288 at M = 17, 27 -> 62 us)
@pytest.mark.parametrize("K,N,G", [(65536, 288, 256), (34816, 512, 32), (12288, 4096, 128)])
@pytest.mark.parametrize("M", [17, 33, 64])
def test_long_rows_are_split(record, K, N, G, M):
    call = dict(op="gemm", M=M, K=K, N=N, G=G, gidx=False)
    r, null = record([call, dict(call, ws=None)])
    kernels = [l["kernel"].split("<")[0] for l in r["launches"]]
    assert kernels == ["k_wide", "k_splitk_reduce"] and launches.outside(r) == []
    assert null["status"] == _abi.ERR_WORKSPACE  # as documented: M > 16 and K >= N


def test_short_rows_keep_their_pair(record):
    """GPTQ-layout weights of G = 32 under X as it is: the pair by bytes (1024 x
    10368 at M = 33 14 us; two row tiles, one workgroup per CU, 21)."""
    calls = [dict(op="gemm", M=M, K=K, N=N, G=32, layout="gptq", gidx=False)
             for K, N, M in ((1024, 10368, 33), (384, 6912, 48), (512, 7680, 65))]
    for r in record(calls):
        assert [mt for mt, _, _, _ in _ordered(r)] == [1]


# ... and over many columns the row groups ran four rounds of one workgroup per CU
# (640 x 28672 at M = 48, 9.6 -> 21.9 us)
@pytest.mark.parametrize("K,N,G,M", [(640, 28672, 128, 48), (1016, 30480, 32, 33), (1536, 27136, 64, 64)])
def test_many_columns_take_the_wide_kernel(record, K, N, G, M):
    r, r17 = record([dict(op="gemm", M=m, K=K, N=N, G=G, gidx=False) for m in (M, 17)])
    assert [l["kernel"].split("<")[0] for l in r["launches"]] == ["k_wide"] and launches.outside(r) == []
    assert len(_ordered(r17)) == 1


# exact tiles cost more the smaller the group
@pytest.mark.parametrize("K,N,G,dtype,M,kernel", [
    (6144, 6144, 32, "bf16", 200, "k_prefill<1, 8, 4"),    # row groups 80 us, 64-row tiles 49
    (3584, 8192, 64, "fp16", 200, "k_prefill<2, 8, 4"),    # 47, 32
    (6144, 6144, 128, "fp16", 100, "k_ordered"),              # 22, 27
    (53248, 2048, 64, "fp16", 160, "k_prefill<2, 8, 4"),   # 128-row tiles 79, 64-row ones 68
    (8192, 28672, 128, "fp16", 128, "k_prefill<4, 8, 8"),  # 77, 85
])
def test_tiles_by_group_size(record, K, N, G, dtype, M, kernel):
    (r,) = record([dict(op="gemm", M=M, K=K, N=N, G=G, dtype=dtype, gidx=False)])
    names = [l["kernel"] for l in r["launches"]]
    assert any(n.startswith(kernel) for n in names), names


# act-order above 64 rows: two launches of the decode kernels cost less than
# dequantizing a small layer (1512 x 3208 at M = 65, 17.4 -> 24.7 us)
@pytest.mark.parametrize("K,N,M,dense", [(1512, 3208, 65, False), (1216, 1968, 65, False), (1216, 1968, 250, True),
                                         (6144, 6144, 100, True), (256, 256, 257, True)])
@pytest.mark.parametrize("layout", ["tiled", "gptq"])
def test_small_act_order_layers(record, K, N, M, dense, layout):
    calls = [dict(op="gemm", M=M, K=K, N=N, path="actorder", layout=layout, ws=ws) for ws in ("doc", "2doc")]
    for r in record(calls):
        assert any("k_dequant16" in l["kernel"] for l in r["launches"]) == dense
        assert any("k_rowmeta" in l["kernel"] for l in r["launches"]) != dense
        assert launches.outside(r) == []
