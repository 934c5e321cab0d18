"""The library's internal matrix-product launches, called directly with a tile and a number of K slices of the
test's choice (csrc/prefill.h declares them; the mangled names are the C++ ABI's)."""
import ctypes

RESID, SWIGLU, PARTIAL, LOGITS, LOGITS_SPLIT = 1, 2, 3, 4, 5  # GemmEpi
# kTiles: rows and columns
TILES = [(32, 128), (64, 128), (128, 128), (128, 256), (128, 256), (256, 128), (256, 160), (256, 224), (256, 256)]
# those that are built for an epilogue (has_tile)
BUILT = {RESID: range(9), SWIGLU: range(9), PARTIAL: range(9), LOGITS: range(6), LOGITS_SPLIT: range(1, 9)}
HEAD_CHUNK = 256  # kHeadChunk
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


def launch_head_logits(lib, x, gain, w, rows, n, k, eps, a, scale, y, err, stream, tile=-1):
    """hipError_t of kf::launch_head_logits: x fp32 or bf16 rows, a [2 HEAD_CHUNK][k] fp16, scale 12 bytes a row of a."""
    f = lib._ZN2kf18launch_head_logitsEPKviPKtS3_iiifPtPdPfPiP12ihipStream_ti
    p, i = ctypes.c_void_p, ctypes.c_int
    f.restype, f.argtypes = i, [p, i, p, p, i, i, i, ctypes.c_float, p, p, p, p, p, i]
    at = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    return f(at(x), x.element_size() == 2, at(gain), at(w), rows, n, k, eps, at(a), at(scale), at(y), at(err), stream, tile)
