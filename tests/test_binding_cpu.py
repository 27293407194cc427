"""What the Python binding does with the library's return codes (no GPU: a
stand-in for the library counts the calls)."""
import pytest
import torch

from paper_2609_03905_amd import ea


class _Library:
    """Returns the given codes of the run entries in turn; planning succeeds
    and asks for a workspace of ``need`` bytes."""

    def __init__(self, codes, need=0):
        self.codes, self.need, self.calls = list(codes), need, []

    def ea_joinagg(self, *a):
        self.calls.append(("run", a[7], a[8]))
        return self.codes.pop(0)

    def ea_joinagg_workspace(self, *a):
        self.calls.append(("plan",))
        a[7]._obj.value = self.need
        return ea.OK

    def ea_repartition_ex(self, *a):
        self.calls.append(("run",))
        return self.codes.pop(0)

    def ea_repartition_plan(self, *a):
        self.calls.append(("plan",))
        return ea.OK

    def ea_last_error(self):
        return b"stand-in"


def _relations():
    p = [[0, 8], [0, 8]]
    return [ea.Relation((8, 8), "f32", p, allocate=False) for _ in range(3)]


def _calls(monkeypatch, codes, entry, need=0, workspace=None):
    a, b, c = _relations()
    fake = _Library(codes, need)
    with monkeypatch.context() as m:
        m.setattr(ea, "lib", lambda: fake)
        try:
            if entry == "joinagg":
                ea.joinagg("ij,jk->ik", ea.JOIN_MUL, ea.AGG_SUM, [a, b], c, stream=0, workspace=workspace)
            else:
                ea.repartition(a, b, stream=0)
            return fake.calls, None
        except ea.EAError as e:
            return fake.calls, e.code


@pytest.mark.parametrize("entry", ["joinagg", "repartition"])
@pytest.mark.parametrize("code", [-8, -7, -6, -2])
def test_an_error_is_raised_and_the_call_made_once(monkeypatch, entry, code):
    # -8: the launch reported an error, its kernels may be queued: a second
    # run would do the work twice, and hide the error if it went through
    calls, raised = _calls(monkeypatch, [code, ea.OK], entry)
    assert raised == code and [c[0] for c in calls] == ["run"]


@pytest.mark.parametrize("entry", ["joinagg", "repartition"])
def test_a_missing_plan_is_made(monkeypatch, entry):
    calls, raised = _calls(monkeypatch, [-9, ea.OK], entry)
    assert raised is None and [c[0] for c in calls] == ["run", "plan", "run"]
    calls, raised = _calls(monkeypatch, [-9, -8], entry)
    assert raised == -8 and [c[0] for c in calls] == ["run", "plan", "run"]


@pytest.mark.parametrize("code,given", [(-1, False), (-4, True)])
def test_a_missing_or_small_workspace_is_looked_up(monkeypatch, code, given):
    ws = torch.zeros(512, dtype=torch.uint8) if given else None
    calls, raised = _calls(monkeypatch, [code, code], "joinagg", need=512 if given else 0, workspace=ws)
    assert raised == code and [c[0] for c in calls] == ["run", "plan", "run"]
    assert (calls[0][2], calls[2][2]) == ((512, 512) if given else (0, 0))


def test_a_bad_argument_beside_a_workspace_is_raised(monkeypatch):
    calls, raised = _calls(monkeypatch, [-1], "joinagg", workspace=torch.zeros(512, dtype=torch.uint8))
    assert raised == -1 and len(calls) == 1
