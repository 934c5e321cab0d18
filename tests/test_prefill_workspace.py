"""The launch plans, the prefill workspace's sizes and its growth, on the host (csrc/prefill.h declares the entry points; the mangled
names are the C++ ABI's).  Nothing here touches a device: allocations are the test's own."""
import ctypes

import pytest

import synth
from tests import gemm_calls as gc
from tests.gemm_calls import Plan

I64, P = ctypes.c_int64, ctypes.c_void_p
OOM = 2  # hipErrorOutOfMemory


class Args(ctypes.Structure):  # PrefillArgs
    _fields_ = ([(n, ctypes.c_int) for n in ("H", "nq", "nkv", "hd", "F")] + [("eps", ctypes.c_float)] +
                [(n, ctypes.c_int) for n in ("T", "pos0", "user")] +
                [("table", P), ("ppu", ctypes.c_int), ("page_stride", I64), ("cos", P), ("sin", P), ("err", P), ("stream", P)])


class Sizes(ctypes.Structure):
    _fields_ = [(n, I64) for n in ("least", "shorter", "full", "own")]


class Workspace(ctypes.Structure):  # PrefillWorkspace
    _fields_ = [("cap", I64), ("refused", ctypes.c_bool), ("mem", P), ("x", P), ("xn", P), ("part", P), ("part_elems", I64),
                ("qkv", Plan), ("oproj", Plan), ("gateup", Plan), ("down", Plan), ("attn_z", ctypes.c_int),
                ("pending", ctypes.c_int), ("q", P), ("o", P), ("act", P)]


Grow = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(P), I64, P)


@pytest.fixture(scope="module")
def lib():
    from paper_2609_34045_amd import stage
    lib = stage.load_library()
    lib.sizes = lib._ZN2kf13prefill_sizesERKNS_11PrefillArgsE
    lib.sizes.restype, lib.sizes.argtypes = Sizes, [ctypes.POINTER(Args)]
    lib.reserve = lib._ZN2kf15prefill_reserveERNS_16PrefillWorkspaceERKNS_11PrefillArgsEPF10hipError_tPPvlP12ihipStream_tE
    lib.reserve.restype, lib.reserve.argtypes = ctypes.c_int, [ctypes.POINTER(Workspace), ctypes.POINTER(Args), Grow]
    return lib


def args(shape, T, pos0=0):
    return Args(H=shape.hidden, nq=shape.n_q_heads, nkv=shape.n_kv_heads, hd=shape.head_dim, F=shape.ffn, T=T, pos0=pos0)


SHAPES = {n: getattr(synth, n) for n in dir(synth) if n.startswith("SHAPE_")}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_a_chunk_fits_where_a_longer_one_ran(lib, name):
    """Up to 2100 tokens: every size covers what every shorter chunk needs, and the full one what its plans use."""
    shape, least, own = SHAPES[name], 0, 0
    for T in range(1, 2101):
        z = lib.sizes(args(shape, T))
        least, own = max(least, z.least), max(own, z.own)
        assert z.least <= z.shorter <= z.full and z.shorter >= least and z.full >= own, T


def reserve(lib, ws, a, memory):
    """prefill_reserve where the device has `memory` bytes; the error and the sizes asked for."""
    asked = []

    def grow(mem, size, stream):
        asked.append(size)
        if size > memory:
            return OOM
        mem[0] = 1 << 40
        return 0

    return lib.reserve(ws, a, Grow(grow)), asked


def check(lib, ws, a):
    """The layout and the plans keep within the workspace."""
    assert ws.part + ws.part_elems * 4 <= ws.mem + ws.cap
    for p, n in ((ws.qkv, (a.nq + 2 * a.nkv) * a.hd), (ws.oproj, a.H), (ws.down, a.H)):
        assert p.slices >= 1 and (p.slices == 1 and n == a.H or p.slices * a.T * n <= ws.part_elems)
    assert ws.attn_z == 1 or ws.attn_z * a.T * a.nq * (a.hd + 2) <= ws.part_elems


@pytest.mark.parametrize("name,T", [("SHAPE_8B", 2048), ("SHAPE_32B", 1024), ("SHAPE_70B", 2048), ("SHAPE_8B", 300), ("SHAPE_TINY", 40)])
def test_a_chunk_runs_in_the_least_memory(lib, name, T):
    """A device that has not the memory for the plans of every chunk, nor for those that follow, still takes the chunk in
    what the sizing rule asks for; short of that it is refused, and the workspace stays as it was."""
    a = args(SHAPES[name], T, 1000)
    z = lib.sizes(a)
    for memory in (z.full, z.full - 1, z.shorter, z.shorter - 1, z.least, z.least - 1):
        ws = Workspace()
        got, asked = reserve(lib, ws, a, memory)
        if memory < z.least:
            assert got == OOM and not ws.mem and ws.cap == 0 and not ws.refused
            continue
        want = next(s for s in (z.full, z.shorter, z.least) if s <= memory)
        assert got == 0 and ws.cap == want and asked[0] == z.full, memory
        check(lib, ws, a)
        assert ws.refused == (want < z.full)
        # later chunks: nothing more is asked for while the buffer holds what they need
        for t in (T, T // 2, 1):
            b = args(SHAPES[name], t, 1000)
            if lib.sizes(b).least <= ws.cap:
                assert reserve(lib, ws, b, 0) == (0, []), (memory, t)
                check(lib, ws, b)


@pytest.mark.parametrize("epi", [gc.RESID, gc.SWIGLU, gc.PARTIAL, gc.LOGITS, gc.LOGITS_SPLIT])
def test_the_plan_takes_only_tiles_that_are_built(lib, epi):
    for m in range(32, 513, 32):
        for n, k in ((64, 64), (777, 320), (128256, 4096), (151936, 5120)):
            p = gc.plan(lib, epi, m, n, k, 8 * m * n)
            assert p.tile in gc.BUILT[epi] and 1 <= p.slices <= gc.MAX_SLICES, (m, n, k)
