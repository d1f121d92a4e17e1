"""A Solver destroys its context once: when its mesh is refused (the object
under construction is finalised after the error as well), when it is closed
twice, and not at all when the context could not be created.  On the CPU, with
the library's calls replaced."""
import gc

import pytest

from paper_2511_17551_amd import workloads as W


@pytest.fixture
def dgx():
    # (not at import: the library takes the HIP runtime that is loaded first,
    # which has to be torch's where tests on the device follow)
    import torch  # noqa: F401
    from paper_2511_17551_amd import dgx as mod
    return mod


@pytest.fixture
def destroyed(dgx, monkeypatch):
    calls = []
    monkeypatch.setattr(dgx, "dgx_create", lambda cfg, sp, rx: dgx.C.c_void_p(1234))
    monkeypatch.setattr(dgx, "dgx_set_mesh", lambda ctx, mesh: None)
    monkeypatch.setattr(dgx, "dgx_destroy", lambda ctx: calls.append(ctx.value))
    return calls


def refuse(dgx):
    def call(*_):
        raise dgx.DgxError(-1, "refused")
    return call


def test_refused_mesh(dgx, destroyed, monkeypatch):
    monkeypatch.setattr(dgx, "dgx_set_mesh", refuse(dgx))
    with pytest.raises(dgx.DgxError):
        dgx.Solver(W.case_c1(n=2))
    gc.collect()
    assert destroyed == [1234]


def test_closed_twice(dgx, destroyed):
    s = dgx.Solver(W.case_c1(n=2))
    s.close()
    s.close()
    del s
    gc.collect()
    assert destroyed == [1234]


def test_no_context(dgx, destroyed, monkeypatch):
    monkeypatch.setattr(dgx, "dgx_create", refuse(dgx))
    with pytest.raises(dgx.DgxError):
        dgx.Solver(W.case_c1(n=2))
    gc.collect()
    assert destroyed == []
