"""The library's internal C++ functions that tests call directly (by their
mangled names, which libdavet.so exports)."""

import ctypes as C

import torch           # first: the library then uses the HIP runtime torch loads

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

plan_gemm16 = _fn("_ZN5davet11plan_gemm16Eiiib", GemmPlan, _i, _i, _i,
                  C.c_bool)
_launch_gemm16 = _fn(
    "_ZN5davet13launch_gemm16EiiRKNS_8GemmPlanEPKtS4_S4_PviiiiPKiPKfiPfmiP12ihipStream_tPi",
    _i, _i, _i, C.POINTER(GemmPlan), _p, _p, _p, _p, _i, _i, _i, _i, _p, _p, _i,
    _p, C.c_size_t, _i, _p, _p)

gemm16_partial_bound = _fn("_ZN5davet20gemm16_partial_boundEiii", C.c_size_t,
                           _i, _i, _i)

EPI_STORE, EPI_ADD_F32, EPI_SWIGLU = 0, 1, 2


def launch_gemm16(dtype, epi, tile, ksplit, A, B, B2, out, M, N, K, ldc,
                  pos=None, cs=None, rope_cols=0, part=None, overflow=None):
    """One product on torch tensors (None: null), tile and split as given."""
    def ptr(t):
        return None if t is None else t.data_ptr()
    return _launch_gemm16(
        dtype, epi, C.byref(GemmPlan(tile, ksplit)), ptr(A), ptr(B), ptr(B2),
        ptr(out), M, N, K, ldc, ptr(pos), ptr(cs), rope_cols, ptr(part),
        0 if part is None else part.numel() * 4, 0,
        torch.cuda.current_stream().cuda_stream, ptr(overflow))
