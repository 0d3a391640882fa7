"""The row norms of the 16-bit path write 16-bit rows only: an fp32 call is
refused before anything is launched, and not run on half the buffer."""

import ctypes as C

import paper_2608_01821_amd as dv
from internal import launch_final_norm_gather, launch_rmsnorm

DAVET_EDTYPE = -3


def test_fp32_rows_are_refused():
    buf = C.create_string_buffer(4096)         # a packed-batch table of zeros
    for dtype in (dv.DAVET_F32, 7, -1):
        assert launch_rmsnorm(None, 1, 64, None, 1e-5, dtype, None,
                              None) == DAVET_EDTYPE
        assert launch_final_norm_gather(None, buf, None, 1, 64, None, 1e-5,
                                        dtype, None, None) == DAVET_EDTYPE
