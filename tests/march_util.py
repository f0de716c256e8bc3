"""The library's marching plan (host code, no GPU needed)."""
import ctypes

import numpy as np

# the operator, and the residual of FP32 fields, march wherever any kernel does
FP64_SWEEPS, FP32_SWEEPS, OPERATOR, FP64_RESIDUAL = 1, 2, 4, 8
ALL = 15


def march_plan(boxes):
    """(kernels that march, segments [n, 6]: XCD, problem, first block x, y, z,
    blocks along z) of a handle over boxes of these block counts."""
    from paper_1009_0798_amd import _lib
    call = _lib.lib().ohm_march_plan
    call.restype = ctypes.c_int32
    bb = np.ascontiguousarray(boxes, dtype=np.int32).reshape(-1, 3)
    kernels = ctypes.c_int32(-1)
    ptr = bb.ctypes.data_as(ctypes.c_void_p)
    n = call(ptr, len(bb), None, 0, ctypes.byref(kernels))
    segs = np.zeros((n, 6), dtype=np.int32)
    assert call(ptr, len(bb), segs.ctypes.data_as(ctypes.c_void_p), n, ctypes.byref(kernels)) == n
    return kernels.value, segs
