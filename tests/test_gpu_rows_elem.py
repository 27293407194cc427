"""RMSNorm and softmax over rows that no 16-byte vector divides: every share of
wavefronts per row, even and uneven segments, masks and infinities, against the
oracle.

Tolerance: f32 rows as the fp32 path's other tests (1e-5: sums of at most 17000
fp32 terms in parallel partial sums); bf16 outputs against the rounded oracle.
"""
import numpy as np
import pytest

import oracle
import synth
from helpers import assert_close, empty, expected, upload, values
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu

LENGTHS = [1, 7, 63, 511, 513, 2047, 2049, 4095, 4099, 8191, 8193, 16383, 16387]  # the last: the scalar path


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", LENGTHS)
def test_rmsnorm_row_lengths(n, dtype):
    rows = 6  # one and a half row tasks
    x, w = synth.normal((rows, n), 3, dtype=dtype), synth.uniform((n,), 4, 0.5, 1.5, dtype=dtype)
    part = synth.splits(n, 1000) if n % 2 else synth.random_splits(n, 5, np.random.default_rng(1))
    X, W = upload(x, dtype, [[0, rows], part]), upload(w, dtype, [part])
    for store in (ea.STORE_CACHED, ea.STORE_STREAM):
        Y = empty((rows, n), dtype, [[0, rows], part])
        ea.joinagg("tc,c->tc", ea.OP_RMSNORM, ea.AGG_SUM, [X, W], Y, eps=1e-6, store=store)
        ref = oracle.rmsnorm(synth.to_f64(x, dtype), synth.to_f64(w, dtype), 1e-6)
        assert_close(values(Y), expected(ref, dtype), rel_fro=1e-5 if dtype == "f32" else 1e-3, what=f"rmsnorm {n}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n,uneven", [(1, False), (63, True), (511, False), (700, True), (2051, False), (4101, True)])
def test_softmax_row_lengths(n, uneven, causal):
    rng = np.random.default_rng(2)
    pk = synth.random_splits(n, 7, rng) if uneven else synth.splits(n, 500)
    pq = synth.random_splits(n, 3, rng)
    s = synth.normal((1, n, n), 5, 2.0, dtype="f32")
    S, P = upload(s, "f32", [[0, 1], pq, pk]), empty((1, n, n), "f32", [[0, 1], pq, pk])
    ea.joinagg("hqk->hqk", ea.OP_SOFTMAX, ea.AGG_LSE, [S], P, causal=causal)
    got, x = values(P)[0], synth.to_f64(s, "f32")[0]
    if causal:
        x = np.where(np.tri(n, dtype=bool), x, -np.inf)
    e = np.exp(x - x.max(1, keepdims=True))
    assert_close(got, e / e.sum(1, keepdims=True), rel_fro=1e-5, what=f"softmax {n} causal={causal}")
    if causal:
        assert not got[np.triu_indices(n, 1)].any()


def test_softmax_minus_infinities():
    s = synth.normal((1, 5, 701), 6, dtype="f32")
    s[0, 1, :], s[0, 2, :700], s[0, 3, 5] = -np.inf, -np.inf, np.finfo(np.float32).min
    p = [[0, 1], [0, 5], [0, 300, 701]]
    S, P = upload(s, "f32", p), empty((1, 5, 701), "f32", p)
    ea.joinagg("hqk->hqk", ea.OP_SOFTMAX, ea.AGG_LSE, [S], P)
    got = values(P)[0]
    assert not got[1].any()  # a row of -inf: zeros
    assert got[2, 700] == 1.0 and not got[2, :700].any()
    x = synth.to_f64(s, "f32")[0, [0, 3, 4]]
    e = np.exp(x - x.max(1, keepdims=True))
    assert_close(got[[0, 3, 4]], e / e.sum(1, keepdims=True), rel_fro=1e-5, what="finite rows")


# element path on one, four and sixteen wavefronts; vector path with the
# exponentials kept in registers and recomputed
@pytest.mark.parametrize("n,dtype", [(5, "f32"), (701, "f32"), (701, "bf16"), (9001, "f32"), (704, "f32"), (4096, "bf16")])
def test_softmax_nan_scores_stay_nan(n, dtype):
    s = synth.normal((1, 4, n), 7, dtype="f32")
    s[0, 1, :] = np.nan
    s[0, 2, :], s[0, 2, n // 2] = -np.inf, np.nan
    s[0, 0, 0] = np.nan
    p = [[0, 1], [0, 4], [0, n]]
    if dtype == "bf16":
        s = (s.view(np.uint32) >> 16).astype(np.uint16)  # truncated: any values do
    S = upload(s, dtype, p)
    x = synth.to_f64(s, dtype)[0]
    for causal in (False, True):
        P = empty((1, 4, n), dtype, p)
        ea.joinagg("hqk->hqk", ea.OP_SOFTMAX, ea.AGG_LSE, [S], P, causal=causal)
        got = values(P)[0]
        seen = np.tri(4, n, dtype=bool) if causal else np.ones((4, n), bool)
        assert not got[~seen].any()  # masked entries are zeros
        for r in range(3):
            vis, out = x[r, seen[r]], got[r, seen[r]]
            if np.isnan(vis).all():
                assert np.isnan(out).all(), (r, causal)
            elif np.isfinite(np.delete(vis, np.flatnonzero(np.isnan(vis)))).any():
                assert np.isnan(out).all() or not np.isnan(vis).any()  # a NaN term makes the sum one
            elif n == 4096:  # long rows on the vector path: a row without a finite score is NaN throughout
                assert np.isnan(out).all()
            else:  # NaN and -inf only: the NaN stays, -inf gives 0
                np.testing.assert_array_equal(np.isnan(out), np.isnan(vis))
                assert not out[~np.isnan(vis)].any()
        assert np.isfinite(got[3]).all() and abs(got[3].sum() - 1) < 0.05


@pytest.mark.parametrize("n", [513, 767, 769, 1023, 1025])  # one wavefront per row, 12 and 16 elements a lane; scalar
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_rows(n, dtype):
    rows = 4101  # more than 4096, the last row task of one row
    x, w = synth.normal((rows, n), 3, dtype=dtype), synth.uniform((n,), 4, 0.5, 1.5, dtype=dtype)
    part = [[0, rows], [0, n // 2 - 1, n]]
    X, W = upload(x, dtype, part), upload(w, dtype, part[1:])
    Y, P = empty((rows, n), dtype, part), empty((rows, n), dtype, part)
    ea.joinagg("tc,c->tc", ea.OP_RMSNORM, ea.AGG_SUM, [X, W], Y, eps=1e-6)
    ea.joinagg("qk->qk", ea.OP_SOFTMAX, ea.AGG_LSE, [X], P)
    x64 = synth.to_f64(x, dtype)
    tol = 1e-5 if dtype == "f32" else 1e-3
    assert_close(values(Y), expected(oracle.rmsnorm(x64, synth.to_f64(w, dtype), 1e-6), dtype), rel_fro=tol, what="rmsnorm")
    e = np.exp(x64 - x64.max(1, keepdims=True))
    assert_close(values(P), expected(e / e.sum(1, keepdims=True), dtype), rel_fro=tol, what="softmax")
