"""The form queries reject NULL handles and leave their outputs untouched."""
import ctypes as C

from paper_2202_04110_amd import lbp


def test_null_handles():
    out = (C.c_int32 * 2)(5, 6)
    assert lbp._lib.lbp_graph_use_automatic(None, 1) == lbp.LBP_E_INVALID
    assert lbp._lib.lbp_graph_form(None, 4, 1.0, out) == lbp.LBP_E_INVALID
    assert list(out) == [5, 6]
