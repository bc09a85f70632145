"""The in-neighbour map as the binding hands it on: any sequence that int() takes, entry by entry."""
import ctypes as C

import numpy as np
import pytest

from paper_1910_00643_amd import binding as B


@pytest.mark.parametrize("values", [[2, 0, 1], (1, 0), [], np.array([3, 1]), [np.int64(3), 1], [1.7, 2], [2 ** 40, -1],
                                    [True, 0], b"\x01\x02\x00\x00", range(5)])
def test_peer_array_is_int_of_every_entry(values):
    got = B._peer_array(values)
    assert isinstance(got, C.Array) and got._type_ is C.c_int32
    assert list(got) == list((C.c_int32 * len(values))(*[int(v) for v in values]))


def test_no_map():
    assert B._peer_array(None) is None
