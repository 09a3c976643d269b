"""The library's own GEMM plans, for tests that must know which kernel a shape takes: its C++
plan functions called through ctypes (host arithmetic; without a GPU they plan for 256 CUs)."""
import ctypes

from paper_2606_26744_amd import hdf


class GemmPlan(ctypes.Structure):
    """hdf::GemmPlan of kernels.hpp."""
    _fields_ = [("nw", ctypes.c_int), ("splits", ctypes.c_int), ("tn", ctypes.c_int),
                ("nt", ctypes.c_bool), ("bm", ctypes.c_int)]


def _plan(symbol, *args):
    f = getattr(hdf.lib(), symbol)
    f.restype = GemmPlan
    return f(*args)


def gemm_plan(bf16: bool, M: int, N: int, K: int) -> GemmPlan:
    return _plan("_ZN3hdf9gemm_planEbiii", ctypes.c_bool(bf16), M, N, K)


def gemm_plan_shared(M: int, N: int, M2: int, N2: int, K: int) -> GemmPlan:
    return _plan("_ZN3hdf16gemm_plan_sharedEiiiii", M, N, M2, N2, K)


def gemm_gated_plan(M: int, F: int, K: int):
    """The plan, or None where the gate and up product goes through partial sums."""
    f = hdf.lib()["_ZN3hdf15gemm_gated_planEiiiPNS_8GemmPlanE"]
    f.restype = ctypes.c_bool
    p = GemmPlan()
    return p if f(M, F, K, ctypes.byref(p)) else None


def deep_tile(p: GemmPlan):
    """(rows, columns) of a matrix-core bound tile."""
    return p.bm, 128 * p.tn
