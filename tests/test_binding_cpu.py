"""The binding's range arrays: every form that numpy can give them reaches the
library as the same int32 values."""
import numpy as np
import pytest

from paper_2403_01876_amd import dv

FAKE = 1 << 40


def cache(batch):
    return dv.Cache(dv.DV_DENSE, 2, 3, 64, batch, [FAKE], max_seq=100)


def read_only(a):
    a.flags.writeable = False
    return a


@pytest.mark.parametrize("form", [
    lambda v: np.array(v, np.int32),
    lambda v: read_only(np.array(v, np.int32)),
    lambda v: np.array(v, np.int64),
    lambda v: np.array(v, ">i4"),
    lambda v: np.repeat(np.array(v, np.int32), 2)[::2],
    lambda v: np.array(v, np.int32).reshape(2, -1),
    lambda v: np.asfortranarray(np.array([v, v], np.int32))[0],
    lambda v: np.array(v + [7], np.int32),
    lambda v: v,
    lambda v: tuple(v),
], ids=["int32", "read-only", "int64", "big-endian", "strided", "2-D", "column", "longer", "list",
        "tuple"])
def test_range_array_forms(form):
    v = [5, 17, 0, 42]
    keep, addr = dv._i32(form(v), 4)
    assert [int(x) for x in np.ctypeslib.as_array(
        (np.ctypeslib.ctypes.c_int32 * 4).from_address(addr))] == v
    assert dv.dv_packed_bytes(cache(4), 0, 2, None, form(v)) == 2 * 2 * 3 * 64 * 2 * sum(v)
    del keep


def test_short_and_empty_range_arrays_are_refused():
    for a in (np.ones(3, np.int32), np.zeros(0, np.int32), [1, 2]):
        with pytest.raises(ValueError):
            dv.dv_packed_bytes(cache(4), 0, 2, None, a)
