"""Which plan a call gets: the dispatch rules of the host code, without a GPU."""
import ctypes

import pytest

import synth
from helpers import describe
from paper_2609_03905_amd import ea


def _product(spec, ext, block=512, dtype="bf16", out=None, join=ea.JOIN_MUL, agg=ea.AGG_SUM, **kw):
    """The plan of an einsum over letters of the given extents in blocks of
    ``block`` (a number, or one per letter)."""
    part = {x: synth.splits(n, min(n, block.get(x, n) if isinstance(block, dict) else block)) for x, n in ext.items()}
    lhs, rhs = spec.split("->")
    ops = [(tuple(ext[x] for x in s), dtype, [part[x] for x in s]) for s in lhs.split(",")]
    ops.append((tuple(ext[x] for x in rhs), out or dtype, [part[x] for x in rhs]))
    return describe(spec, join, agg, ops, **kw)


@pytest.mark.parametrize("spec,t,j,k,by_class", [
    ("tj,jk,jk->tk", 1792, 8192, 2752, 1), ("tj,jk,jk->tk", 1536, 8192, 3072, 1), ("tj,jk,jk->tk", 1024, 8192, 5504, 1),
    ("tj,jk,jk->tk", 2048, 8192, 2752, 0), ("tj,kj,kj->tk", 2048, 8192, 2752, 0), ("tj,jk,jk->tk", 2048, 8192, 2304, 0),
    ("tj,jk->tk", 2560, 8192, 3584, 1), ("tj,kj->tk", 2304, 6144, 4096, 1),
])
def test_balanced_tiles_are_reordered_only_where_panels_are_saved(spec, t, j, k, by_class):
    d = _product(spec, dict(t=t, j=j, k=k), join=ea.OP_SWIGLU if spec.count("j") == 3 else ea.JOIN_MUL)
    assert (d["kind"], d["balanced"], d["by_class"]) == ("gemm", 1, by_class)


# sizes whose 128-row plan measured slower than 256-row tiles (up to 39%), and
# their neighbours that it serves better
@pytest.mark.parametrize("spec,t,j,k,tile_m", [
    ("tj,jk,jk->tk", 1280, 8192, 15360, 256), ("tj,jk->tk", 6144, 8192, 6200, 256), ("tj,kj->tk", 6144, 8192, 6200, 256),
    ("tj,jk,jk->tk", 5000, 2048, 4096, 256), ("tj,jk->tk", 2304, 2048, 9984, 256), ("tj,kj->tk", 4096, 4096, 5000, 256),
    ("tj,jk,jk->tk", 1000, 4096, 11008, 256), ("tj,jk->tk", 2304, 4096, 15104, 256), ("tj,jk,jk->tk", 1280, 8192, 8832, 256),
    ("tj,jk,jk->tk", 1111, 8192, 8192, 256), ("tj,kj->tk", 3000, 4096, 6400, 256), ("tj,kj->tk", 3000, 4096, 5600, 128),
    ("tj,jk->tk", 2304, 2048, 8192, 128), ("tj,jk->tk", 1000, 4096, 16640, 128), ("tj,jk,jk->tk", 1280, 8192, 6656, 128),
    ("tj,jk->tk", 1024, 4096, 4096, 128), ("tj,jk->tk", 64, 4096, 4096, 128), ("tj,jk->tk", 4096, 4096, 4096, 256),
])
def test_gemm_tile_rows(spec, t, j, k, tile_m):
    d = _product(spec, dict(t=t, j=j, k=k), join=ea.OP_SWIGLU if spec.count("j") == 3 else ea.JOIN_MUL)
    assert (d["kind"], d["tile_m"]) == ("gemm", tile_m)


def test_a_plan_cleared_meanwhile_is_not_recognised():
    # a call finds its plan, the cache is cleared (another thread), then the
    # call would be entered: its plan is gone
    L = ea.lib()
    L.ea_internal_generation.restype = ctypes.c_uint64
    remember = lambda g: L.ea_internal_remember(b"a test's call", ctypes.c_uint64(g))
    found_in = L.ea_internal_generation()
    ea.plan_cache_clear()
    assert remember(found_in) == 0
    assert remember(L.ea_internal_generation()) == 1
    ea.plan_cache_clear()


SUM, MAX, NONE = ea.AGG_SUM, ea.AGG_MAX, ea.AGG_NONE


@pytest.mark.parametrize("i,j,jblock,rows", [
    (1 << 20, 64, 64, 0), (1 << 20, 128, 128, 0), (1 << 20, 256, 256, 1), (1 << 20, 256, 32, 0), (1 << 20, 256, 4, 0),
    (1 << 20, 256, 64, 1), (32768, 64, 64, 0), (32768, 512, 512, 1), (4096, 64, 64, 1), (4096, 2048, 8, 1), (4096, 31, 31, 0),
    (13000, 2048, 63, 1), (100000, 512, 63, 1), (65536, 2048, 8, 0),
])
def test_reduction_lanes(i, j, jblock, rows):
    # a wavefront per output or lanes along the output, whichever measured
    # faster (up to 20 times, with many outputs and short blocks)
    d = _product("ij->i", dict(i=i, j=j), dict(j=jblock), "f32", agg=SUM)
    assert (d["kind"], d["rows"]) == ("reduce", rows)


@pytest.mark.parametrize("block,kind,rounds", [(4, "generic", None), (8, "generic", None), (16, "reduce", 1),
                                               (32, "reduce", 4), (512, "reduce", 4)])
@pytest.mark.parametrize("spec", ["ij->ji", "ij,ij->ij"])
def test_elementwise_rounds_follow_the_blocks(spec, block, kind, rounds):
    d = _product(spec, dict(i=2048, j=2048), block, "f32", agg=NONE)
    assert d["kind"] == kind and d.get("rounds") == rounds


@pytest.mark.parametrize("i,j,dtype", [(1 << 24, 32, "f32"), (1 << 24, 200, "bf16"), (70_000_000, 256, "bf16"),
                                       (70_000_000, 40, "bf16")])
def test_reduction_tables_and_launches_stay_small(i, j, dtype):
    d = _product("ij->i", dict(i=i, j=j), dict(i=1 << 20), dtype, agg=SUM)
    assert d["work"] * d["threads"] < 1 << 32  # what a launch holds
    assert d["table_bytes"] <= i * j * ea.ELEM_SIZE[dtype] // 64  # of the input's bytes


@pytest.mark.parametrize("spec,ext,kind", [
    # no row and no column letter, many small products, products with a vector
    ("ij,ij->i", dict(i=131072, j=64), "reduce"), ("ij,ij->i", dict(i=1 << 20, j=4), "reduce"),
    ("ij,ij->j", dict(i=64, j=131072), "reduce"), ("ij,ij->i", dict(i=3, j=5), "reduce"),
    ("bij,bjk->bik", dict(b=524288, i=2, j=8, k=2), "reduce"), ("bij,bjk->bik", dict(b=65536, i=16, j=2, k=16), "reduce"),
    ("bij,bjk->bik", dict(b=65536, i=4, j=1, k=64), "reduce"), ("ij,j->i", dict(i=1 << 20, j=4), "reduce"),
    ("ij,j->i", dict(i=100, j=8192), "reduce"), ("ij,i->j", dict(i=16, j=1 << 20), "reduce"),
    # matrix products of any size
    ("ij,jk->ik", dict(i=33, j=33, k=33), "contract"), ("ij,jk->ik", dict(i=4096, j=1, k=4096), "contract"),
    ("hqd,hkd->hqk", dict(h=8, q=256, k=256, d=128), "contract"), ("bij,bjk->bik", dict(b=20000, i=16, j=16, k=16), "contract"),
    ("hqd,hkd->hqk", dict(h=4096, q=1, k=256, d=128), "contract"), ("ij,j->i", dict(i=4096, j=4096), "contract"),
])
def test_contraction_or_reduction(spec, ext, kind):
    assert _product(spec, ext, 1 << 30, "f32")["kind"] == kind


@pytest.mark.parametrize("spec,ext,block,kind", [
    ("bij,bjk->bik", dict(b=16384, i=4, j=16, k=4), dict(b=1), "contract"),  # a workgroup per block either way
    ("bij,bjk->bik", dict(b=65536, i=4, j=16, k=4), dict(b=1024), "reduce"),
    ("ij,i->j", dict(i=8192, j=100), dict(i=512), "contract"),                # a long serial sum per lane
    ("ij,j->i", dict(i=1 << 20, j=16), dict(j=8), "reduce"),
])
def test_contraction_or_reduction_in_blocks(spec, ext, block, kind):
    assert _product(spec, ext, block, "f32")["kind"] == kind


@pytest.mark.parametrize("i,j,k,tile", [
    (174, 65, 758, 64), (174, 163, 758, 32), (500, 1001, 500, 32), (1000, 1001, 300, 64), (300, 401, 300, 16), (75, 9, 1116, 16),
    (512, 512, 512, 32), (256, 256, 256, 16), (1024, 128, 1024, 64),
])
def test_contraction_tiles_read_along_k(i, j, k, tile):
    # odd j: every load of a small tile touches as many cache lines as rows
    assert _product("ij,kj->ik", dict(i=i, j=j, k=k), 1 << 30, "f32")["tile"] == tile


@pytest.mark.parametrize("spec,ext,block,kind", [
    ("ij,jk->ik", dict(i=40000, j=16000, k=64), 1 << 30, "gemm32"),  # an operand block of 2.4 GiB
    ("ij,kj->ik", dict(i=64, j=16000, k=40000), 1 << 30, "gemm32"),
    ("ij,jk->ik", dict(i=65536, j=64, k=65536), 1 << 30, "gemm32"),  # an output block of 2^32 elements
    ("ij,jk->ik", dict(i=40000, j=13000, k=64), 1 << 30, "contract"),
    ("ij,jk->ik", dict(i=131072, j=4096, k=65536), 4096, "contract"),  # 2^21 tiles of 64 x 64
])
def test_large_f32_products(spec, ext, block, kind):
    assert _product(spec, ext, block, "f32")["kind"] == kind


def _rows(op, rows, n, dtype, nseg=1):
    part = [[0, rows], synth.splits(n, -(-n // nseg))]
    if op == "rmsnorm":
        return describe("tc,c->tc", ea.OP_RMSNORM, ea.AGG_SUM,
                        [((rows, n), dtype, part), ((n,), dtype, part[1:]), ((rows, n), dtype, part)], eps=1e-6)
    return describe("qk->qk", ea.OP_SOFTMAX, ea.AGG_LSE, [((rows, n), dtype, part)] * 2)


@pytest.mark.parametrize("op,rows,n,dtype,path,waves,per_lane", [
    ("rmsnorm", 262144, 33, "bf16", "scalar", None, None), ("rmsnorm", 64, 383, "f32", "scalar", None, None),
    ("rmsnorm", 32768, 385, "bf16", "elem", 1, 8), ("rmsnorm", 32768, 515, "bf16", "elem", 1, 12),
    ("rmsnorm", 32768, 1023, "f32", "elem", 1, 16), ("rmsnorm", 1024, 515, "bf16", "elem", 4, 8),
    ("rmsnorm", 32768, 1031, "bf16", "scalar", None, None), ("rmsnorm", 32768, 1031, "f32", "elem", 4, 8),
    ("rmsnorm", 1024, 1031, "bf16", "elem", 4, 8), ("rmsnorm", 32768, 1501, "bf16", "elem", 4, 8),
    ("softmax", 262144, 33, "bf16", "elem", 1, 8), ("softmax", 32768, 700, "bf16", "elem", 1, 12),
    ("softmax", 4096, 700, "bf16", "elem", 4, 8), ("softmax", 32768, 1030, "bf16", "elem", 4, 8),
    ("softmax", 100, 8193, "f32", "elem", 16, 16), ("softmax", 100, 16385, "f32", "scalar", None, None),
    ("rmsnorm", 32768, 1024, "bf16", "vec", None, None),
])
def test_row_paths(op, rows, n, dtype, path, waves, per_lane):
    d = _rows(op, rows, n, dtype)
    assert (d["kind"], d["path"]) == (op, path)
    if path == "elem":
        assert (d["waves"], d["per_lane"]) == (waves, per_lane)


@pytest.mark.parametrize("rows,n,nseg,path", [
    (65536, 60, 60, "elem"), (65536, 33, 2, "elem"), (65536, 33, 1, "scalar"), (32768, 1201, 2, "scalar"), (32768, 1031, 3, "scalar"),
    (32768, 1031, 5, "elem"), (32768, 1401, 3, "elem"),
])
def test_rmsnorm_in_segments(rows, n, nseg, path):
    # the scalar path walks the segments one after the other
    assert _rows("rmsnorm", rows, n, "bf16", nseg)["path"] == path


@pytest.mark.parametrize("rows,n", [(17_000_000, 2051), (17_000_000, 515), (5_000_000, 9001)])
def test_row_launches_hold_every_row(rows, n):
    # rows of a workgroup or of sixteen wavefronts each: more threads than a
    # launch holds take the scalar path, four rows per workgroup
    d = _rows("rmsnorm", rows, n, "f32")
    assert d["work"] * d["threads"] < 1 << 32


def test_tables_of_layouts_and_calls_are_bounded_and_given_back():
    L = ea.lib()
    L.ea_internal_table_bytes.restype = ctypes.c_int64
    n, bound = 100_000, 64 << 20
    nb, splits, h = (ctypes.c_int32 * 1)(n), (ctypes.c_int64 * (n + 1))(*range(n + 1)), ctypes.c_void_p()
    ids = 0
    for i in range(200):  # 160 MB of split points in all
        splits[n] = n + i
        assert L.ea_relation_create(1, (ctypes.c_int64 * 1)(n + i), 0, nb, splits, None, 0, ctypes.byref(h)) == 0
        L.ea_relation_destroy(h)
        ids = max(ids, L.ea_internal_table_bytes())
    assert 8 * n < ids <= 2 * bound
    L.ea_internal_generation.restype = ctypes.c_uint64
    for i in range(2000):  # 200 MB of call keys
        assert L.ea_internal_remember(b"%099999d" % i, ctypes.c_uint64(L.ea_internal_generation())) == 1
    assert L.ea_internal_table_bytes() <= 2 * bound
    ea.plan_cache_clear()
    assert L.ea_internal_table_bytes() == 0


@pytest.mark.parametrize("spec,ext,block,dtype", [
    ("ij,jk->ik", dict(i=1024, j=1024, k=1024), 16, "f32"), ("ij,jk->ik", dict(i=2048, j=2048, k=2048), 16, "bf16"),
])
def test_tuple_records_are_made_on_the_device(spec, ext, block, dtype):
    # a record of 64 or 72 bytes per tuple beside the join's own 8 or 12: in
    # device memory alone, not in the image that the host builds and uploads
    d = _product(spec, ext, block, dtype, agg=SUM)
    tuples = 1
    for n in ext.values():
        tuples *= n // block
    assert d["kind"] in ("contract", "gemm")
    assert d["table_bytes"] >= 64 * tuples and d["host_bytes"] < 40 * tuples
