"""The library's choice of kernel for a projection: its planner is host code, called by its C++ name."""
import ctypes as C

import paper_2512_20276_amd as af

EPI_STORE, EPI_STORE_F32, EPI_RESID, EPI_SWIGLU, EPI_QKV = range(5)


class TilePlan(C.Structure):
    _fields_ = [("fm", C.c_int), ("splits", C.c_int), ("wg", C.c_int)]


class StreamPlan(C.Structure):
    _fields_ = [("fm", C.c_int), ("cb", C.c_int), ("splits", C.c_int)]


_tile = af.lib["_ZN2af9tile_planEiii"]
_tile.restype, _tile.argtypes = TilePlan, [C.c_int] * 3
_f32_small = af.lib["_ZN2af14gemm_f32_smallEiii"]
_f32_small.restype, _f32_small.argtypes = C.c_bool, [C.c_int] * 3
_stream = af.lib["_ZN2af11stream_planEiiiiRKNS_8TilePlanEPNS_10StreamPlanE"]
_stream.restype, _stream.argtypes = C.c_bool, [C.c_int] * 4 + [C.POINTER(TilePlan), C.POINTER(StreamPlan)]


def padk(k):
    """K as the packed weights hold it."""
    return (k + 255) // 256 * 256


def tile_plan(M, N, K):
    return _tile(M, N, padk(K))


def f32_small(M, N, K):
    """Whether an fp32 projection runs on the 16 x 32 tiles."""
    return _f32_small(M, N, padk(K))


def stream_plan(epi, M, N, K):
    """(row blocks, column blocks, K splits) of the streaming kernel, or None where the tiles run."""
    p = StreamPlan()
    t = tile_plan(M, N, K)
    return (p.fm, p.cb, p.splits) if _stream(M, N, padk(K), epi, C.byref(t), C.byref(p)) else None
