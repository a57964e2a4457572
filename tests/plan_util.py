"""The library's planner of projection launches, asked without a device."""
import ctypes
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2405_16444_amd", "libcacheblend.so")
SEG, SWIGLU, F32 = 0, 1, 2
_fn = []


def projection_plan(epi, rows, n, k, hl=0, raw=0, w8=0, scratch=2 ** 64 - 1):
    """The plan of a bf16 problem with enough scratch: `rows` x k times n columns (SWIGLU: of gate and of up) of which the first hl take
    operand pairs; raw: a deviation is wanted.  tile: rows x columns (gate and up together)."""
    if not _fn:
        if not os.path.exists(LIB):
            from paper_2405_16444_amd import build
            build.build()
        import torch  # noqa: F401  (the library uses the HIP runtime that torch brings)
        fn = ctypes.CDLL(LIB).cb_internal_projection_plan
        fn.argtypes = [ctypes.c_int] * 8 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
        fn.restype = ctypes.c_size_t
        _fn.append(fn)
    out = (ctypes.c_int * 8)()
    parked = _fn[0](1, epi, rows, n, k, hl, raw, w8, scratch, out)
    plan = dict(zip(("kind", "bm", "bn", "splits", "shared", "mode", "stagger", "finish"), out), parked=parked)
    plan["tile"] = (plan["bm"], plan["bn"])
    return plan
