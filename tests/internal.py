"""The library's internal C++ functions that tests call directly (by their
mangled names, which libdavet.so exports)."""

import ctypes as C

import paper_2608_01821_amd as dv

_L = dv.raw()


class GemmPlan(C.Structure):
    _fields_ = [("tile", C.c_int), ("ksplit", C.c_int)]


def _fn(name, restype, *argtypes):
    f = _L[name]
    f.restype, f.argtypes = restype, argtypes
    return f


_p, _i, _f = C.c_void_p, C.c_int, C.c_float

launch_rmsnorm = _fn(
    "_ZN5davet14launch_rmsnormEPKfiiS1_fiPvP12ihipStream_t",
    _i, _p, _i, _i, _p, _f, _i, _p, _p)
launch_final_norm_gather = _fn(
    "_ZN5davet24launch_final_norm_gatherEPKfRKNS_7SeqPackEPKiiiS1_fiPvP12ihipStream_t",
    _i, _p, _p, _p, _i, _i, _p, _f, _i, _p, _p)
