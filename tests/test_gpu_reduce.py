"""The reduction and elementwise kernel (einsums of one or two inputs, at most
one contracted letter): orders, aggregations, both lane layouts and every
share of wavefronts per output, against the oracle's fp64 einsum.

Tolerance: sums of at most 5000 fp32 terms of N(0,1) data in parallel partial
sums differ from fp64 by well under 1e-5 of their norm; maxima, sums of small
integers and elementwise joins of them are exact.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_close, describe, empty, expected, upload, values
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu

JOIN = {"mul": (ea.JOIN_MUL, oracle.JOIN_MUL), "add": (ea.JOIN_ADD, oracle.JOIN_ADD)}
AGG = {"none": (ea.AGG_NONE, oracle.AGG_NONE), "sum": (ea.AGG_SUM, oracle.AGG_SUM), "max": (ea.AGG_MAX, oracle.AGG_MAX)}


def _run(spec, join, agg, ext, nblocks=3, dtype="f32", out="f32", integers=False, residual=False):
    rng = np.random.default_rng(11)
    lhs, rhs = spec.split("->")
    ops = lhs.split(",")
    part = {x: synth.random_splits(n, nblocks, rng) for x, n in ext.items()}
    shape = lambda s: tuple(ext[x] for x in s)
    draw = (lambda s, i: synth.integers(shape(s), 80 + i, -3, 3, dtype)) if integers else \
        (lambda s, i: synth.normal(shape(s), 80 + i, dtype=dtype))
    xs = [draw(s, i) for i, s in enumerate(ops)]
    ins = [upload(x, dtype, [part[c] for c in s]) for x, s in zip(xs, ops)]
    C = empty(shape(rhs), out, [part[c] for c in rhs])
    R = r = None
    if residual:
        r = synth.integers(shape(rhs), 90, -3, 3, out)
        R = upload(r, out, [part[c] for c in rhs])
    ea.joinagg(spec, JOIN[join][0], AGG[agg][0], ins, C, residual=R)
    ref = oracle.einsum(spec, [synth.to_f64(x, dtype) for x in xs], JOIN[join][1], AGG[agg][1])
    return values(C), ref + synth.to_f64(r, out) if residual else ref


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("spec,join,agg", [
    ("ij->i", "mul", "sum"), ("ij->i", "add", "max"), ("ij->j", "mul", "sum"), ("ij->j", "mul", "max"),
    ("ijk->ik", "mul", "sum"), ("ijk->ki", "mul", "max"), ("kij->ij", "mul", "sum"), ("ij->ji", "mul", "none"),
    ("abcd->dbca", "add", "none"), ("ij,ij->ij", "mul", "none"), ("ij,ji->ij", "add", "none"),
    ("ij,j->ij", "mul", "none"), ("i,j->ji", "add", "none"), ("ij,ij->i", "mul", "max"), ("ij,jk->ik", "mul", "max"),
    ("ij,kj->ik", "add", "sum"), ("ij,j->i", "add", "max"),
])
def test_orders_exact_on_integers(spec, join, agg, dtype):
    ext = dict(i=37, j=45, k=19, a=3, b=5, c=7, d=4)
    got, ref = _run(spec, join, agg, {x: ext[x] for x in spec if x in ext}, dtype=dtype, integers=True)
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("agg", ["sum", "max"])
@pytest.mark.parametrize("spec", ["ij->i", "ij->j"])
@pytest.mark.parametrize("i,j", [(1, 1), (31, 33), (64, 31), (200, 255), (33, 5000), (5000, 33), (4097, 70), (70, 4097)])
def test_lengths(spec, agg, i, j):
    got, ref = _run(spec, "mul", agg, dict(i=i, j=j), nblocks=1 if min(i, j) < 3 else 5)
    assert_close(got, expected(ref, "f32"), rel_fro=1e-5, what=f"{spec} {agg} {i} {j}")


@pytest.mark.parametrize("n", [33000, 140000, 1100000])  # 4 and 1 wavefronts per 64 outputs; several per thread
def test_many_outputs(n):
    for spec, ext in (("ij->j", dict(i=40, j=n)), ("j,j->j", dict(j=n))):
        agg = "sum" if "i" in spec else "none"
        got, ref = _run(spec, "add", agg, ext, integers=True, dtype="bf16")
        np.testing.assert_array_equal(got, ref)


def test_residual_and_output_types():
    for out in ("f32", "bf16", "f16"):
        got, ref = _run("ij->i", "mul", "sum", dict(i=33, j=70), integers=True, residual=True, out=out)
        np.testing.assert_array_equal(got, expected(ref, out))


def test_infinities_nan_and_signed_zeros():
    x = np.array([[-np.inf, -np.inf], [np.nan, 1.0], [-0.0, -0.0], [np.inf, -np.inf]], np.float32)
    X = upload(x, "f32", [[0, 4], [0, 2]])
    M, S = empty((4,), "f32", [[0, 4]]), empty((4,), "f32", [[0, 4]])
    ea.joinagg("ij->i", ea.JOIN_MUL, ea.AGG_MAX, [X], M)
    ea.joinagg("ij->i", ea.JOIN_MUL, ea.AGG_SUM, [X], S)
    np.testing.assert_array_equal(values(M), [-np.inf, 1.0, 0.0, np.inf])  # a maximum passes a NaN over
    np.testing.assert_array_equal(values(S), [-np.inf, np.nan, 0.0, np.nan])
    Y = empty((2, 4), "f32", [[0, 2], [0, 4]])
    ea.joinagg("ij->ji", ea.JOIN_MUL, ea.AGG_NONE, [X], Y)  # a transpose keeps every bit
    torch.cuda.synchronize()
    assert Y.bytes().cpu().numpy().tobytes() == np.ascontiguousarray(x.T).tobytes()


# several rows per wavefront; four wavefronts per 64 rows, once and several times over
@pytest.mark.parametrize("i,j", [(131077, 203), (20001, 70), (1048583, 33)])
def test_many_rows(i, j):
    x = synth.integers((i, j), 5, -3, 3, "bf16")
    pi = [0, i // 3, i // 3 + 1, i]
    for part in ([0, j], [0, j // 2, j]):
        X, S, M = upload(x, "bf16", [pi, part]), empty((i,), "f32", [pi]), empty((i,), "f32", [pi])
        ea.joinagg("ij->i", ea.JOIN_MUL, ea.AGG_SUM, [X], S)
        ea.joinagg("ij->i", ea.JOIN_MUL, ea.AGG_MAX, [X], M)
        ref = synth.to_f64(x, "bf16")
        np.testing.assert_array_equal(values(S), ref.sum(1))
        np.testing.assert_array_equal(values(M), ref.max(1))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("spec,ext", [
    ("ij,ij->i", dict(i=37, j=45)), ("ij,ij->j", dict(i=37, j=45)), ("bji,ijb->bi", dict(b=3, i=70, j=33)),
    ("ij,ij->i", dict(i=300, j=513)), ("bij,bjk->bik", dict(b=3000, i=2, j=3, k=2)), ("ij,j->i", dict(i=20000, j=3)),
])
def test_sums_of_products_that_no_tile_serves(spec, ext, dtype):
    # no row and no column letter, many small products, products with a vector
    part = {x: synth.splits(n, n) for x, n in ext.items()}
    ops = [(tuple(ext[x] for x in s), dtype, [part[x] for x in s]) for s in spec.replace("->", ",").split(",")]
    assert describe(spec, ea.JOIN_MUL, ea.AGG_SUM, ops)["kind"] == "reduce"
    for nblocks in (1, 3):
        got, ref = _run(spec, "mul", "sum", ext, nblocks if min(ext.values()) >= nblocks else 1, dtype, integers=True)
        np.testing.assert_array_equal(got, ref)
