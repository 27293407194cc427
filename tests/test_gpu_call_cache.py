"""Repeated calls skip validation and planning: what a call depends on must all
be part of what it is recognised by, and what is not (data pointers) must be
looked at every time."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_close, empty, expected, upload, values
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu


def _rms(x, w, eps, part):
    X, W = upload(x, "f32", [[0, x.shape[0]], part]), upload(w, "f32", [part])
    Y = ea.Relation(x.shape, "f32", [[0, x.shape[0]], part])
    for _ in range(2):
        ea.joinagg("tc,c->tc", ea.OP_RMSNORM, ea.AGG_SUM, [X, W], Y, eps=eps)
    return Y.bytes().cpu().numpy().tobytes()


def test_parameters_layouts_and_data_are_all_seen():
    x, w = synth.normal((8, 64), 1, dtype="f32"), synth.normal((64,), 2, dtype="f32")
    a = _rms(x, w, 1e-6, [0, 64])
    assert _rms(x, w, 10.0, [0, 64]) != a          # another eps, same layouts
    assert _rms(x, w, 1e-6, [0, 32, 64]) != a      # another partition, same shape
    y = np.ascontiguousarray(x[:, ::-1])           # other data
    got = np.frombuffer(_rms(y, w, 1e-6, [0, 64]), np.float32).reshape(8, 64)
    ref = oracle.rmsnorm(y.astype(np.float64), w.astype(np.float64), 1e-6)
    assert np.linalg.norm(got - ref) < 1e-6 * np.linalg.norm(ref)
    assert _rms(x, w, 1e-6, [0, 64]) == a


def test_data_pointers_are_read_on_every_call():
    # inputs, residual and output moved to other buffers between two recognised
    # calls: the second result goes to the new output, the first stays
    p = [[0, 64], [0, 64]]
    xs = [synth.integers((64, 64), i, -3, 3, "f32") for i in range(6)]
    run = lambda: ea.joinagg("ij,jk->ik", ea.JOIN_MUL, ea.AGG_SUM, [A, B], C, residual=R)
    A, B, R = (upload(x, "f32", p) for x in xs[:3])
    C = empty((64, 64), "f32", p)
    run()
    run()
    first, old = values(C), C.data
    np.testing.assert_array_equal(first, xs[0].astype(np.float64) @ xs[1] + xs[2])
    moved = [upload(x, "f32", p) for x in xs[3:]] + [empty((64, 64), "f32", p)]
    keep = []  # the old buffers, so that their addresses are not handed out again
    for rel, new in zip((A, B, R, C), moved):
        assert ea.lib().ea_relation_set_data(rel.handle, new.data.data_ptr(), new.data.numel()) == ea.OK
        keep.append(rel.data)
        rel.data = new.data
    run()
    np.testing.assert_array_equal(values(C), xs[3].astype(np.float64) @ xs[4] + xs[5])
    C.data = old
    np.testing.assert_array_equal(values(C), first)


def test_attention_parameters_separate_calls():
    # the same relations under another scale, mask, list of sequences or
    # grouping: each call against its own, and again in the other order
    S, part = 384, [[0, 1], [0, 1, 2], [0, 128, 256, 384], [0, 128]]
    q, k, v = (synth.normal((1, 2, S, 128), i, dtype="bf16") for i in (1, 2, 3))
    Q, K, V = (upload(x, "bf16", part) for x in (q, k, v))
    calls = [dict(scale=0.08), dict(scale=0.02), dict(scale=0.08, causal=True), dict(scale=0.08, seq_ends=[128, 384]),
             dict(scale=0.08, seq_ends=[256, 384]), dict(scale=0.08, causal=True, seq_ends=[256, 384])]
    first = {}
    for order in (range(6), reversed(range(6))):
        for i in order:
            c = calls[i]
            O = empty((1, 2, S, 128), "bf16", part)
            ea.joinagg("bhqd,bhkd,bhkd->bhqd", ea.OP_ATTENTION, ea.AGG_LSE, [Q, K, V], O, **c)
            got, ends, lo = values(O), c.get("seq_ends", [S]), 0
            for hi in ends:
                ref = oracle.attention(*(synth.to_f64(x[:, :, lo:hi], "bf16") for x in (q, k, v)), c.get("causal", False),
                                       c["scale"])
                assert_close(got[:, :, lo:hi], expected(ref, "bf16"), what=str(c))
                lo = hi
            assert np.array_equal(first.setdefault(i, got), got)
    # two query heads over one key/value head: other relations for K and V, one
    # grouping parameter apart from a call that is refused
    g = [[0, 1], [0, 1], part[2], part[3]]
    K1, V1 = upload(k[:, :1], "bf16", g), upload(v[:, :1], "bf16", g)
    O = empty((1, 2, S, 128), "bf16", part)
    run = lambda **kw: ea.joinagg("bhqd,bgkd,bgkd->bhqd", ea.OP_ATTENTION, ea.AGG_LSE, [Q, K1, V1], O, scale=0.08, **kw)
    for _ in range(2):
        run(gqa_group=2)
        with pytest.raises(ea.EAError):
            run()
    rep = [synth.to_f64(np.repeat(x[:, :1], 2, 1), "bf16") for x in (k, v)]
    assert_close(values(O), expected(oracle.attention(synth.to_f64(q, "bf16"), *rep, False, 0.08), "bf16"), what="gqa")


def test_residual_layouts_separate_calls():
    # with and without a residual, and with one of another partition (refused)
    p = [[0, 64], [0, 96]]
    a, r = synth.integers((64, 96), 1, -3, 3, "f32"), synth.integers((64, 96), 2, -3, 3, "f32")
    A, R, other = upload(a, "f32", p), upload(r, "f32", p), upload(r, "f32", [[0, 32, 64], [0, 96]])
    C = empty((64, 96), "f32", p)
    run = lambda res: ea.joinagg("ij->ij", ea.JOIN_MUL, ea.AGG_NONE, [A], C, residual=res)
    for _ in range(2):
        run(None)
        np.testing.assert_array_equal(values(C), a)
        run(R)
        np.testing.assert_array_equal(values(C), a.astype(np.float64) + r)
        with pytest.raises(ea.EAError):
            run(other)


def test_two_threads_on_the_table_of_calls():
    # both threads make calls that are new to the table and calls known to it,
    # each on its own stream and relations
    p = lambda n: [[0, n], [0, 64]]
    done, errors = [], []

    def work(t):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for i in range(40):
                    n = 64 + 8 * (i % 10) + (t if i % 2 else 0)  # half of the layouts are common
                    x = synth.integers((n, 64), 100 * t + i, -3, 3, "f32")
                    X, Y = upload(x, "f32", p(n)), ea.Relation((n,), "f32", [[0, n]])
                    ea.joinagg("ij->i", ea.JOIN_MUL, ea.AGG_SUM, [X], Y)
                    s.synchronize()
                    got = Y.bytes().view(torch.float32).cpu().numpy()
                    np.testing.assert_array_equal(got, x.sum(1))
            done.append(t)
        except BaseException as e:  # noqa: BLE001  (reported below)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors and sorted(done) == [0, 1], errors


def test_invalid_calls_stay_invalid_after_valid_ones():
    p = [[0, 128], [0, 128]]
    A, B = (upload(synth.normal((128, 128), i, dtype="f32"), "f32", p) for i in (1, 2))
    C = ea.Relation((128, 128), "f32", p)
    run = lambda ins, out, **kw: ea.joinagg("ij,jk->ik", ea.JOIN_MUL, ea.AGG_SUM, ins, out, **kw)
    for _ in range(2):
        run([A, B], C)
    none = ea.Relation((128, 128), "f32", p, allocate=False)
    for ins, out, kw, code in [([A, none], C, {}, -1), ([A, B], none, {}, -1), ([A, B], C, dict(residual=none), -1),
                               ([A, B], C, dict(store=7), -1), ([A, B], C, dict(gqa_group=-1), -1),
                               ([A, ea.Relation((128, 128), "f32", [[0, 64, 128], [0, 128]])], C, {}, -6)]:
        for _ in range(2):
            with pytest.raises(ea.EAError) as e:
                run(ins, out, **kw)
            assert e.value.code == code
    run([A, B], C)
    ea.plan_cache_clear()  # the recognised calls point into the plans
    assert ea.plan_cache_size() == 0
    prm, _ = ea._params()
    handles = (ctypes.c_void_p * 2)(A.handle.value, B.handle.value)
    assert ea.lib().ea_joinagg(b"ij,jk->ik", ea.JOIN_MUL, ea.AGG_SUM, 2, handles, C.handle, ctypes.byref(prm), None, 0,
                               None) == -9  # not planned any more
    run([A, B], C)


def test_workspace_grows_for_a_larger_plan_on_the_same_stream():
    s = torch.cuda.Stream()
    outs = []
    with torch.cuda.stream(s):
        for t in (128, 256, 128):  # split sums: partials in the stream's workspace
            x, w = synth.integers((t, 4096), t, -2, 2, "bf16"), synth.integers((4096, 256), 3, -2, 2, "bf16")
            X, W = upload(x, "bf16", [[0, t], [0, 4096]]), upload(w, "bf16", [[0, 4096], [0, 256]])
            Y = ea.Relation((t, 256), "f32", [[0, t], [0, 256]])
            ea.joinagg("tj,jk->tk", ea.JOIN_MUL, ea.AGG_SUM, [X, W], Y)
            outs.append((Y, synth.to_f64(x, "bf16") @ synth.to_f64(w, "bf16")))
    s.synchronize()
    for Y, ref in outs:
        np.testing.assert_array_equal(Y.bytes().view(torch.float32).cpu().numpy().reshape(ref.shape), ref)
