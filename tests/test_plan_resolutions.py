"""The resolutions a Plan takes: lists of pairs of whole numbers by the direct route, all else as numpy converts it; both give the
numbers that numpy gives, and refuse what it refuses."""
import numpy as np
import pytest

from paper_2501_09253_amd.binding import Plan


@pytest.mark.parametrize("res", [[(16, 24)], ([8, 8], (3, 5)), [(np.int64(7), True), (-1, 0)], np.array([[1, 2], [3, 4]]),
                                 [1, 2, 3, 4], [(1.5, 2)], [[(1, 2), (3, 4)]], [(2**31 - 1, -2**31)], [], [np.array([5, 6])],
                                 (2**31, 1), [(2**31, 1)], [(1, -2**31 - 1)], [(1, 2, 3)], [(1, 2), (3,)], [("a", 1)], [(1, None)]])
def test_same_as_numpy(res):
    try:
        want = np.asarray(res, dtype=np.int32).reshape(-1, 2)
    except Exception as e:
        with pytest.raises(type(e)):
            Plan._flat(res)
        return
    got = Plan._flat(res)
    assert got.itemsize == 4 and got.tolist() == want.reshape(-1).tolist()


def test_no_request_is_refused():
    from paper_2501_09253_amd import PserveError
    with pytest.raises((PserveError, RuntimeError)):
        Plan([])
