"""Block-GEMM tile heights (128 and 256 rows) and partial K steps.

Contracted block extents that are no multiple of 32 end in a partial 32-deep
step on the direct-load kernels.  Integer data: any summation order is exact,
so every plan gives the oracle's bits.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from helpers import assert_close, empty, expected, upload, values
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu


def _product(spec, T, K, pt, pj, pk, dtype="bf16", out="f32", seed=3, residual=False, data=None):
    J = pj[-1]
    kmajor = "kj" in spec
    sw = spec.count("j") == 3
    x = data[0] if data else synth.integers((T, J), seed, -2, 2, dtype)
    ws = [data[1]] if data else [synth.integers((K, J) if kmajor else (J, K), seed + 1 + i, -2, 2, dtype)
                                 for i in range(1 + sw)]
    X = upload(x, dtype, [pt, pj])
    Ws = [upload(w, dtype, [pk, pj] if kmajor else [pj, pk]) for w in ws]
    Y = empty((T, K), out, [pt, pk])
    R = r = None
    if residual:
        r = synth.integers((T, K), seed + 9, -4, 4, out)
        R = upload(r, out, [pt, pk])
    ea.joinagg(spec, ea.OP_SWIGLU if sw else ea.JOIN_MUL, ea.AGG_SUM, [X] + Ws, Y, residual=R)
    fx = synth.to_f64(x, dtype)
    p = [fx @ (synth.to_f64(w, dtype).T if kmajor else synth.to_f64(w, dtype)) for w in ws]
    if sw:
        return values(Y), p[0] / (1.0 + np.exp(-p[0])) * p[1]
    return values(Y), p[0] + synth.to_f64(r, out) if residual else p[0]


@pytest.fixture(params=["128", "256"])
def tile_rows(request, monkeypatch):
    monkeypatch.setenv("EA_GEMM_TILE_M", request.param)
    ea.plan_cache_clear()
    yield request.param
    ea.plan_cache_clear()


@pytest.mark.parametrize("spec", ["tj,jk->tk", "tj,kj->tk"])
@pytest.mark.parametrize("pj", [
    [0, 8], [0, 24], [0, 32, 40], [0, 8, 48, 120, 128, 200],   # one partial step; a partial step in every block
    [0, 64, 96, 136, 392],                                      # more steps than stages, tails in the middle
    [0, 2744],
], ids=str)
def test_partial_k_steps(tile_rows, spec, pj):
    T, K = 141, 264  # ragged rows and columns of either tile
    got, ref = _product(spec, T, K, [0, 128, T], pj, [0, 8, K])
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("spec", ["tj,jk,jk->tk", "tj,kj,kj->tk"])
@pytest.mark.parametrize("pj", [[0, 40], [0, 96, 200]], ids=str)
def test_partial_k_steps_swiglu(tile_rows, spec, pj):
    got, ref = _product(spec, 141, 136, [0, 141], pj, [0, 64, 136])
    assert_close(got, ref, rel_fro=1e-5, what=spec)  # fp32 exp and reciprocal: about 1e-6


@pytest.mark.parametrize("dtype,out", [("bf16", "bf16"), ("f16", "f16"), ("f16", "f32")])
def test_tiles_residual(tile_rows, dtype, out):
    got, ref = _product("tj,jk->tk", 200, 392, [0, 200], [0, 64, 136], [0, 256, 392], dtype, out, residual=True)
    np.testing.assert_array_equal(got, expected(ref, out))


@pytest.mark.parametrize("T,J,K", [(64, 4096, 256), (130, 2048, 384), (8, 1000, 8)])
def test_tiles_split_sums(tile_rows, T, J, K):
    # few output tiles: each one's K walk is cut into runs that workgroups merge
    got, ref = _product("tj,jk->tk", T, K, [0, T], synth.splits(J, 512), [0, K])
    np.testing.assert_array_equal(got, ref)


def test_partial_steps_non_finite(tile_rows):
    # masked lanes of a partial step load the block's first values: a NaN or an
    # infinity there must reach its own row and column only
    T, J, K = 70, 40, 72
    x, w = synth.normal((T, J), 1, dtype="f16"), synth.normal((J, K), 2, dtype="f16")
    x.view(np.float16)[0, 0] = np.nan
    w.view(np.float16)[0, 0] = np.inf
    got, _ = _product("tj,jk->tk", T, K, [0, T], [0, J], [0, K], "f16", data=(x, w))
    assert np.isnan(got[0]).all()
    assert not np.isfinite(got[1:, 0]).any()
    assert np.isfinite(got[1:, 1:]).all()


def test_more_tuples_than_the_direct_kernels_hold():
    # 130 contracted blocks per output block: the register-staged kernel
    got, ref = _product("tj,jk->tk", 70, 72, [0, 70], list(range(0, 1041, 8)), [0, 72])
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("spec,T,J,pk", [
    ("tj,jk,jk->tk", 400, 2048, [0, 512, 1024, 1536, 2048, 2560, 2904]),  # 46 tiles in 3 classes: 16, 15, 15
    ("tj,jk->tk", 400, 8192, [0, 520, 1024, 2792]),                       # panels shared in block order: kept
    ("tj,kj->tk", 700, 8192, [0, 1000, 2048]),                            # the same
    ("tj,kj->tk", 700, 8192, [0, 1000, 1408]),                            # three tile rows: half a stripe
    ("tj,jk->tk", 700, 4096, [0, 512, 1024, 1152]),                       # 256 x 128 tiles, an odd number of columns
    ("tj,kj->tk", 520, 2000, [0, 3000]),                                  # runs in no common step: block order
], ids=str)
def test_balanced_runs(monkeypatch, spec, T, J, pk):
    # equal runs of K steps, the tiles in block order or ordered for the runs that walk K together
    monkeypatch.setenv("EA_GEMM_TILE_M", "256")
    monkeypatch.setenv("EA_GEMM_SCHEDULE", "balanced")
    ea.plan_cache_clear()
    try:
        got, ref = _product(spec, T, pk[-1], [0, 256, T], synth.splits(J, 512), pk)
    finally:
        ea.plan_cache_clear()
    if spec.count("j") == 3:
        assert_close(got, ref, rel_fro=1e-5, what=spec)
    else:
        np.testing.assert_array_equal(got, ref)
