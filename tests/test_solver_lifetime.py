"""A Solver destroys its context once: when its mesh is refused (the object
under construction is finalised after the error as well), when it is closed
twice, and not at all when the context could not be created.  On the CPU, with
the library's calls replaced."""
import gc

import pytest

from paper_2511_17551_amd import dgx
from paper_2511_17551_amd import workloads as W


@pytest.fixture
def destroyed(monkeypatch):
    calls = []
    monkeypatch.setattr(dgx, "dgx_create", lambda cfg, sp, rx: dgx.C.c_void_p(1234))
    monkeypatch.setattr(dgx, "dgx_set_mesh", lambda ctx, mesh: None)
    monkeypatch.setattr(dgx, "dgx_destroy", lambda ctx: calls.append(ctx.value))
    return calls


def refuse(*_):
    raise dgx.DgxError(-1, "refused")


def test_refused_mesh(destroyed, monkeypatch):
    monkeypatch.setattr(dgx, "dgx_set_mesh", refuse)
    with pytest.raises(dgx.DgxError):
        dgx.Solver(W.case_c1(n=2))
    gc.collect()
    assert destroyed == [1234]


def test_closed_twice(destroyed):
    s = dgx.Solver(W.case_c1(n=2))
    s.close()
    s.close()
    del s
    gc.collect()
    assert destroyed == [1234]


def test_no_context(destroyed, monkeypatch):
    monkeypatch.setattr(dgx, "dgx_create", refuse)
    with pytest.raises(dgx.DgxError):
        dgx.Solver(W.case_c1(n=2))
    gc.collect()
    assert destroyed == []
