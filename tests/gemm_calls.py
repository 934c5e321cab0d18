"""The library's internal matrix-product launches, called directly with a tile and a number of K slices of the
test's choice (csrc/prefill.h declares them; the mangled names are the C++ ABI's)."""
import ctypes

RESID, SWIGLU, PARTIAL, LOGITS, LOGITS_SPLIT = 1, 2, 3, 4, 5  # GemmEpi
TILES = 9  # kTiles
MAX_SLICES = 8  # kGemmMaxSlices


class Plan(ctypes.Structure):
    _fields_ = [("tile", ctypes.c_int), ("slices", ctypes.c_int)]


def plan(lib, epi, m, n, k, part_elems=0):
    f = lib._ZN2kf9gemm_planEiiiil
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 4 + [ctypes.c_int64]
    return f(epi, m, n, k, part_elems)


def launch_gemm(lib, epi, tile, slices, a, w, w2, m, n, k, c, cb, err, stream):
    """hipError_t of kf::launch_gemm; the operands are tensors or None."""
    f = lib._ZN2kf11launch_gemmEiRKNS_8GemmPlanEPKtS4_S4_iiiPfPtPiP12ihipStream_t
    p = ctypes.c_void_p
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.POINTER(Plan), p, p, p] + [ctypes.c_int] * 3 + [p] * 4
    at = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    return f(epi, ctypes.byref(Plan(tile, slices)), at(a), at(w), at(w2), m, n, k, at(c), at(cb), at(err), stream)
