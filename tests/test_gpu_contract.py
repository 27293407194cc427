"""The two-operand contraction kernels: every letter order they accept, each
output tile (16, 32, 64), ragged blocks, vector and element loads, against the
oracle's fp64 einsum.

Tolerance: fp32 products and sums of K terms differ from fp64 by at most about
K/2 * 2^-24 of the sum of absolute products; with N(0,1) data that is under
1e-5 of the output's norm for K <= 300 (bf16 and f16 inputs widen exactly).
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from helpers import assert_close, describe, empty, expected, upload, values
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu


def _run(spec, ext, nblocks, dtype="f32", out="f32", residual=False, inputs=None):
    rng = np.random.default_rng(7)
    lhs, rhs = spec.split("->")
    ops = lhs.split(",")
    part = {x: synth.random_splits(n, nblocks, rng) for x, n in ext.items()}
    shape = lambda s: tuple(ext[x] for x in s)
    xs = inputs or [synth.normal(shape(s), 60 + i, dtype=dtype) for i, s in enumerate(ops)]
    ins = [upload(x, dtype, [part[c] for c in s]) for x, s in zip(xs, ops)]
    C = empty(shape(rhs), out, [part[c] for c in rhs])
    R = r = None
    if residual:
        r = synth.normal(shape(rhs), 69, dtype=out)
        R = upload(r, out, [part[c] for c in rhs])
    ea.joinagg(spec, ea.JOIN_MUL, ea.AGG_SUM, ins, C, residual=R)
    ref = oracle.einsum(spec, [synth.to_f64(x, dtype) for x in xs], oracle.JOIN_MUL, oracle.AGG_SUM)
    if residual:
        ref = ref + synth.to_f64(r, out)
    return values(C), ref


SPECS = ["ij,jk->ik", "ij,kj->ik", "ji,jk->ik", "ji,kj->ik", "ij,jk->ki", "hij,hkj->hik", "hij,hjk->hik",
         "ijh,hjk->ikh", "abij,abjk->aibk", "ij,j->i", "j,jk->k"]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("spec", SPECS)
def test_contract_letter_orders(spec, dtype):
    # odd extents: element loads along every letter, ragged tails of every tile
    ext = dict(i=67, j=45, k=33, h=3, a=2, b=3)
    got, ref = _run(spec, {x: ext[x] for x in spec if x in ext}, 2, dtype)
    assert_close(got, ref, rel_fro=1e-5, what=f"{spec} {dtype}")


@pytest.mark.parametrize("i,j,k", [
    (1, 1, 1), (16, 4, 16), (17, 3, 15), (64, 128, 64), (65, 260, 130), (512, 96, 448), (500, 100, 444),
    (1024, 64, 1024), (1000, 36, 1060), (1031, 33, 1025),
])
@pytest.mark.parametrize("spec", ["ij,jk->ik", "ij,kj->ik", "ji,jk->ik"])
def test_contract_tiles(spec, i, j, k):
    got, ref = _run(spec, dict(i=i, j=j, k=k), 1 if min(i, j, k) < 3 else 3)
    assert_close(got, ref, rel_fro=1e-5, what=f"{spec} {i} {j} {k}")


@pytest.mark.parametrize("dtype,out", [("f32", "bf16"), ("f32", "f16"), ("bf16", "bf16"), ("f16", "f32")])
def test_contract_residual_and_output_types(dtype, out):
    got, ref = _run("ij,jk->ik", dict(i=70, j=51, k=37), 2, dtype, out, residual=True)
    assert_close(got, expected(ref, out), rel_fro=1e-5 if out == "f32" else 1e-3, what=f"{dtype} {out}")


@pytest.mark.parametrize("n", [33, 1030])
def test_contract_non_finite_inputs_stay_in_their_rows(n):
    # the kernels pad rows and the contracted letter: nothing outside the
    # row of A (column of B) that holds it may see a NaN or an infinity
    a = synth.normal((n, 37), 1, dtype="f32")
    b = synth.normal((37, n), 2, dtype="f32")
    a[n - 1, 36], a[0, 0], b[36, n - 1] = np.inf, np.nan, np.inf
    got, _ = _run("ij,jk->ik", dict(i=n, j=37, k=n), 2, inputs=[a, b])
    with np.errstate(invalid="ignore"):
        ref = a.astype(np.float64) @ b.astype(np.float64)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    np.testing.assert_array_equal(np.isposinf(got), np.isposinf(ref))
    ok = np.isfinite(ref)
    assert_close(got[ok], ref[ok], rel_fro=1e-5, what="finite part")


@pytest.mark.parametrize("i,j,k,tile", [
    (64, 128, 64, 16), (65, 131, 40, 16),      # vectors; element loads along j, odd rows
    (512, 512, 512, 32), (516, 1000, 444, 32), (600, 300, 517, 32),
    (1024, 64, 1024, 64), (1031, 33, 1025, 64), (1030, 70, 1100, 64),
])
@pytest.mark.parametrize("spec", ["ij,jk->ik", "ij,kj->ik", "ji,jk->ik", "ji,kj->ik"])
def test_contract_every_tile(spec, i, j, k, tile):
    # the sizes' tiles are what the plans take (two blocks along j)
    ext, part = dict(i=i, j=j, k=k), dict(i=[0, i], j=[0, j // 8 * 4, j], k=[0, k])
    lhs, rhs = spec.split("->")
    shape, parts = (lambda s: tuple(ext[x] for x in s)), (lambda s: [part[x] for x in s])
    ops = [(shape(s), "f32", parts(s)) for s in lhs.split(",") + [rhs]]
    assert describe(spec, ea.JOIN_MUL, ea.AGG_SUM, ops)["tile"] == tile
    xs = [synth.normal(s, 40 + n, dtype="f32") for n, (s, _, _) in enumerate(ops[:2])]
    ins = [upload(x, "f32", p) for x, (_, _, p) in zip(xs, ops)]
    C = empty((i, k), "f32", parts(rhs))
    ea.joinagg(spec, ea.JOIN_MUL, ea.AGG_SUM, ins, C)
    a, b = (synth.to_f64(x, "f32") for x in xs)
    assert_close(values(C), (a if spec[0] == "i" else a.T) @ (b if spec[3] == "j" else b.T), rel_fro=1e-5,
                 what=f"{spec} {i} {j} {k}")
