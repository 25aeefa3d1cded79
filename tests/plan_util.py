"""Which kernel each product of a layer call takes, by the library's own dispatch (moe_test_plan, host only)."""
import ctypes

from paper_2201_05596_amd import binding as B

F32_KERNELS = ["none", "rows16", "rows32", "rows_split8", "rows_split4", "tile_narrow", "tile", "split1", "split2", "ffn"]


def plan(T, d, f, E, k, C, residual=False, packed=False):
    """([expert GEMM-1, expert GEMM-2, dense GEMM-1, dense GEMM-2], [first, second half shared]); codes as in csrc/api.hip and, of the tiled
    kernels, at tgemm_code in csrc/moe_internal.h."""
    shape = B.make_shape(T, d, f, E, k, C, "bf16", residual, B.MOE_FLAG_PACKED_WEIGHTS if packed else 0)
    kernels, shared = (ctypes.c_int32 * 4)(), (ctypes.c_int32 * 2)()
    assert B.load_library().moe_test_plan(ctypes.byref(shape), kernels, shared) == 0
    return list(kernels), list(shared)


def plan_f32(T, d, f, E, k, C, residual=False):
    """Names (F32Kernel in csrc/moe_internal.h) for the experts' products and, with a dense branch, for its."""
    shape, kernels = B.make_shape(T, d, f, E, k, C, "f32", residual), (ctypes.c_int32 * 4)()
    assert B.load_library().moe_test_plan(ctypes.byref(shape), kernels, (ctypes.c_int32 * 2)()) == 0
    return [F32_KERNELS[n] for n in kernels][:4 if residual else 2]
