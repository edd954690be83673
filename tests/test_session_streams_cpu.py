"""Stream opening and closing through the native module against the C calls
through ctypes, argument form by argument form."""
import ctypes as C

import numpy as np
import pytest

import paper_2608_06146_amd as pa
from paper_2608_06146_amd import _lib

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
