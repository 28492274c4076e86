"""A batch's number of operators is bounded by memory alone: 2^24 of them are looked at, and refused only for
what they are (here NULL, so nothing touches a GPU)."""
import ctypes as C

import paper_2402_09531_amd as dw


def test_count_has_no_bound_of_its_own():
    n = 1 << 24
    h = C.c_void_p()
    st = dw.lib().dwfmm_batch_create((C.c_void_p * n)(), n, 0, None, C.byref(h))
    assert st == dw.E_INVALID and dw.lib().dwfmm_last_error() == b"ops contains NULL"
