"""Stream opening and closing through the native module against the C calls
through ctypes, argument form by argument form."""
import ctypes as C
import os
import sys

import numpy as np
import pytest

import paper_2608_06146_amd as pa
from paper_2608_06146_amd import _lib, build

FORMS = [(-1, 0), (0, 0), (np.int64(0), np.int32(3)), (0.9, "4"), (True, False), (2**32 - 1, 0), (2**32, 2**33 + 5),
         (-(2**70) - 1, 0), (0, 6), (0, -1), (7, 0), (-2, 0), (None, 0), (0, None), ("x", 0), (float("nan"), 0)]


def twin():
    s = pa.DecodeSession(4, 1, 64, 64)
    s.open()
    s.prepare([5], [0])
    s.commit()
    return s


def ctypes_open(s, parent, fork):
    i = C.c_int32(0)
    _lib.check(_lib.lib().padoc_session_open(s.handle, int(parent), int(fork), C.byref(i)))
    return i.value


def outcome(f, *a):
    try:
        return f(*a)
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)


@pytest.mark.parametrize("parent,fork", FORMS)
def test_open_close_as_ctypes(parent, fork):
    a, b = twin(), twin()
    n = a.n_open
    x, y = outcome(a.open, parent, fork), outcome(ctypes_open, b, parent, fork)
    assert x == y
    assert a.n_open == n + (not isinstance(x, tuple))
    va, vb = a.view(), b.view()
    assert np.array_equal(va["seg"], vb["seg"]) and np.array_equal(va["row_id"], vb["row_id"])
    for i in (parent, x if isinstance(x, int) else 0):
        n = a.n_open
        r = outcome(a.close, i)
        assert r == outcome(lambda i: _lib.check(_lib.lib().padoc_session_close(b.handle, int(i))), i)
        assert a.n_open == n - (r is None)
    assert np.array_equal(a.view()["row_id"], b.view()["row_id"])


def test_destroyed_and_prepared():
    s = twin()
    s.prepare([1], [1])
    with pytest.raises(pa.PadocError, match="has not been launched"):
        s.open()
    with pytest.raises(pa.PadocError, match="has not been launched"):
        s.close(0)
    s.commit()
    assert s.open(parent=0, fork=6) == 1 and s.close(stream_id=1) is None
    s.destroy()
    for f in (s.open, lambda: s.close(0)):
        with pytest.raises(ValueError, match="session is closed"):
            f()


# ---------------------------------------------------------------- without the module

@pytest.fixture
def no_module(monkeypatch):
    """An interpreter that the native module was not built for."""
    monkeypatch.setitem(sys.modules, "paper_2608_06146_amd._streams", None)
    monkeypatch.setattr(_lib, "_lib", None)


def test_the_library_loads_without_the_module(no_module):
    plan = pa.TreePlan(pa.segments_layout([(-1, 0, 10, 10)], 0), 2, 1, 64, "bf16", 0, num_kv_rows=10, num_q_rows=10)
    assert plan.export()["work"].size and isinstance(twin()._streams, _lib.CtypesStreams)


@pytest.mark.parametrize("parent,fork", FORMS)
def test_open_close_without_the_module(no_module, parent, fork):
    test_open_close_as_ctypes(parent, fork)
    test_destroyed_and_prepared()


@pytest.fixture
def built(monkeypatch, tmp_path):
    """build() of the present objects into another folder."""
    if not os.path.exists(build.LIB):
        pytest.skip("nothing is built")
    for name in ("LIB", "STREAMS"):
        monkeypatch.setattr(build, name, str(tmp_path / os.path.basename(getattr(build, name))))
    return tmp_path


def test_build_without_python_headers(built, monkeypatch):
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(built)})
    (built / os.path.basename(build.STREAMS)).write_text("old")
    build.build(force=False)
    assert os.path.exists(build.LIB) and not os.path.exists(build.STREAMS)


def test_failed_build_replaces_nothing(built, monkeypatch):
    bad = built / "bad.cpp"
    bad.write_text("#error no\n")
    monkeypatch.setattr(build, "STREAMS_SOURCE", str(bad))
    with pytest.raises(RuntimeError, match="compile failed"):
        build.build(force=False)
    assert not os.path.exists(build.LIB) and not os.path.exists(build.STREAMS)
