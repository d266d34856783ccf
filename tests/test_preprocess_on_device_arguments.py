"""Arguments that smat_preprocess refuses are refused by smat_preprocess_on_device in the same way, without a look at what they do not name."""
import ctypes

import numpy as np
import pytest

import paper_2408_11551_amd as S
from paper_2408_11551_amd import smat as binding


@pytest.mark.parametrize("M,K", [(1 << 40, 4), ((1 << 31) - 16, 4), (-1, 4), (4, 1 << 24), (4, -1)])
def test_sizes_out_of_range(M, K):
    # (one page, and row_ptr[M] far behind it)
    row_ptr = np.zeros(512, np.int64)
    never = binding._ScratchFn(lambda *_: None)
    for dtype in (0, 4, 7):
        got = []
        for call, extra in ((binding._lib.smat_preprocess, ()), (binding._lib.smat_preprocess_on_device, (never, None))):
            out = ctypes.c_void_p()
            got.append((call(M, K, row_ptr.ctypes.data, None, None, dtype, None, *extra, ctypes.byref(out)), S.smat_last_error()))
            assert out.value is None
        assert got[0] == got[1] and got[0][0] in (1, 3)


@pytest.mark.parametrize("ptr,columns,what", [
    ([1, 2, 3], [0, 1, 2], "ptr[0]"), ([0, 2, 1], [0, 1, 2], "decreases"), ([0, 2, 3], [0, 1, 2], "lengths"), ([0, 1, 3], [0, 2, 2], "ascend"),
    ([0, 1, 3], [0, 2, 1], "ascend"), ([0, 1, 2], [0, 5], "below")])
def test_patterns_that_are_none(ptr, columns, what):
    ptr, columns = np.array(ptr, np.uint32), np.array(columns, np.uint32)
    pairs, count = np.empty(64, np.int32), ctypes.c_int64()
    # (an address that is never used: patterns are looked at first)
    status = binding._lib.smat_pattern_partners(2, 5, ptr.ctypes.data, columns.ctypes.data, 300, 1 << 20, 1 << 20, None, pairs.ctypes.data, 32, ctypes.byref(count))
    assert status == 1 and what in S.smat_last_error()
