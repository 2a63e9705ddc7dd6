"""The largest cells are limits of the interface: calls beyond them are refused
before any device call, with a message that names the limit and no other cause
(FP64 cells somewhat above it would fit the LDS)."""
import ctypes as C
import threading

import pytest

from paper_2507_21239_amd import _lib
from paper_2507_21239_amd import workloads as W


@pytest.mark.parametrize("schedule", ["plain", "batched"])
@pytest.mark.parametrize("precision,largest", [("fp64", 1536), ("mixed", 2048)])
def test_cells_beyond_the_limit_are_refused_by_its_name(precision, largest, schedule):
    lib = _lib.load()
    got = []

    def call():   # the message of a context-free call belongs to its thread
        buf = C.create_string_buffer(64)
        at = C.addressof(buf)
        params = _lib.make_params(W.benchmark_params(), precision, schedule)
        parts = _lib.Particles(4, 0, 0, at, at, 0, None)
        cells = _lib.Cells(1, largest + 1, at, at, at)
        st = lib.mcd_collide_noalloc(C.byref(params), C.byref(parts), C.byref(cells), 0.0, 1, 0, None, None)
        got.append((st, lib.mcd_last_error(None).decode()))
    t = threading.Thread(target=call)
    t.start()
    t.join()
    st, msg = got[0]
    assert st == -1 and str(largest) in msg and "LDS" not in msg
