"""Edge validation in pieces over several host threads: the first bad edge of
the call is the one named, wherever the pieces' edges lie, before any device
call."""
import ctypes

import numpy as np
import pytest


def _build(evq, V, base, dels, adds):
    arr = (evq.Batch * 1)()
    ptr = lambda x: x.ctypes.data_as(ctypes.POINTER(evq.Edge)) if len(x) else None
    arr[0] = evq.Batch(ptr(dels), len(dels), ptr(adds), len(adds))
    h = ctypes.c_void_p()
    rc = evq.lib.evq_build(V, ptr(base), len(base), arr, 1, None, None, ctypes.byref(h))
    assert not h.value
    return rc


@pytest.mark.parametrize("where,at,field,value,msg", [
    ("base", 131071, 0, 1000, "out of range at index 131071"),
    ("base", 131072, 1, 1000, "out of range at index 131072"),
    ("base", 399999, 2, 0, "zero weight at index 399999"),
    ("dels", 0, 1, 4294967295, "batch deletions"),
    ("adds", 140000, 2, 0, "zero weight at index 140000"),
])
def test_first_bad_edge_is_named(where, at, field, value, msg):
    import paper_2502_10579_amd as evq
    parts = {k: np.ones((n, 3), np.uint32) for k, n in (("base", 400000), ("dels", 131073), ("adds", 150000))}
    parts[where][at, field] = value
    parts["adds"][149999, 0] = 5000  # a later one, in the last piece
    assert _build(evq, 1000, parts["base"], parts["dels"], parts["adds"]) == evq.EVQ_EINVAL
    assert msg in evq.last_error(), evq.last_error()


@pytest.mark.parametrize("bad,msg", [(None, "batch deletions is NULL"), ("base", "base: zero weight at index 199999"),
                                     ("adds", "batch deletions is NULL")])
def test_null_span_is_named_in_its_turn(bad, msg):
    import paper_2502_10579_amd as evq
    parts = {k: np.ones((n, 3), np.uint32) for k, n in (("base", 200000), ("adds", 10))}
    if bad:
        parts[bad][-1, 2] = 0
    arr = (evq.Batch * 1)()
    ptr = lambda x: x.ctypes.data_as(ctypes.POINTER(evq.Edge))
    arr[0] = evq.Batch(None, 7, ptr(parts["adds"]), 10)
    h = ctypes.c_void_p()
    rc = evq.lib.evq_build(1000, ptr(parts["base"]), len(parts["base"]), arr, 1, None, None, ctypes.byref(h))
    assert rc == evq.EVQ_EINVAL and not h.value
    assert msg in evq.last_error(), evq.last_error()
