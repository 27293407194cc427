"""Repeated calls skip validation and planning: what a call depends on must all
be part of what it is recognised by, and what is not (data pointers) must be
looked at every time."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from helpers import upload
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
    assert _rms(2.0 * x, w, 1e-6, [0, 64]) is not None
    assert _rms(x, w, 1e-6, [0, 64]) == a


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
