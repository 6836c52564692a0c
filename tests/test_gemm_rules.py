"""Which tiles a bf16 GEMM of many rows runs on: the library's own rules, asked on the CPU.

The expected sides are those measured faster on one MI355X (by 5% or more, with
weights from HBM); the figures are beside the rules in gemm_wide.hip.  A call
that the 256-row tiles cannot take as it is stays with the others."""
import ctypes as C

import pytest

STORE, SILU, LOGITS = 0, 2, 3


class Seg(C.Structure):
    _fields_ = [("w", C.c_void_p), ("n0", C.c_int), ("n", C.c_int)]


class GemmArgs(C.Structure):
    _fields_ = [("x", C.c_void_p), ("ldx", C.c_int), ("M", C.c_int), ("seg", Seg * 3), ("nseg", C.c_int), ("N", C.c_int),
                ("K", C.c_int), ("splits", C.c_int), ("y", C.c_void_p), ("ldy", C.c_int), ("split_stride", C.c_longlong),
                ("tilemax", C.c_void_p), ("ntiles", C.c_int), ("tilekey", C.c_void_p), ("mode", C.c_int),
                ("summed", C.c_int), ("accumulate", C.c_int)]


@pytest.fixture(scope="module")
def rules():
    import paper_2607_20791_amd as rgd

    def fn(name):
        f = getattr(rgd.lib, "_ZN3rgd%d%sERKNS_8GemmArgsE" % (len(name), name))
        f.restype, f.argtypes = C.c_bool, [C.POINTER(GemmArgs)]
        return lambda a: f(C.byref(a))
    return {n: fn(n) for n in ("gemm_wide_fits", "gemm_wide_wins", "gemm_sums_splits")}


def _args(mode, N, K, M, splits=1, nseg=1):
    a = GemmArgs(x=1 << 20, ldx=K, M=M, nseg=nseg, N=N, K=K, splits=splits, y=1 << 30, ldy=N, mode=mode)
    a.seg[0].n = N
    return a


def _side(rules, a):
    if rules["gemm_sums_splits"](a):
        return "sum"
    return "wide" if rules["gemm_wide_fits"](a) and rules["gemm_wide_wins"](a) else "narrow"


@pytest.mark.parametrize("mode,N,K,splits,M,side", [
    # LM head: one round of 128-row workgroups beats one of 256-row ones, and three beat two at K = 4096
    (LOGITS, 32000, 4096, 1, 130, "narrow"), (LOGITS, 32000, 4096, 1, 256, "narrow"), (LOGITS, 65536, 2048, 1, 256, "narrow"),
    (LOGITS, 32000, 4096, 1, 512, "narrow"), (LOGITS, 32000, 4096, 1, 600, "wide"), (LOGITS, 65536, 4096, 1, 257, "wide"),
    (LOGITS, 66308, 128, 1, 130, "wide"), (LOGITS, 65476, 1024, 1, 300, "wide"), (LOGITS, 66048, 1024, 1, 130, "wide"), (LOGITS, 128256, 1024, 1, 130, "wide"), (LOGITS, 128256, 4096, 1, 256, "wide"),
    (LOGITS, 128256, 4096, 1, 257, "narrow"), (LOGITS, 128256, 4096, 1, 400, "wide"), (LOGITS, 128256, 4096, 1, 128, "narrow"),
    # SwiGLU: a second round for 257 to 384 rows does not pay
    (SILU, 3584, 1024, 1, 130, "wide"), (SILU, 14336, 4096, 1, 256, "wide"), (SILU, 14336, 4096, 1, 300, "wide"),
    (SILU, 10752, 3072, 1, 300, "narrow"), (SILU, 10752, 3072, 1, 400, "wide"), (SILU, 14336, 4096, 1, 100, "narrow"),
    # projections: few steps per split, few workgroups
    (STORE, 1536, 1024, 4, 300, "narrow"), (STORE, 1536, 1024, 4, 640, "narrow"), (STORE, 1024, 1024, 4, 1024, "narrow"),
    (STORE, 1024, 3584, 8, 257, "narrow"), (STORE, 1024, 3584, 8, 640, "wide"), (STORE, 3072, 2048, 8, 257, "narrow"),
    (STORE, 6144, 4096, 4, 300, "wide"), (STORE, 4096, 14336, 8, 256, "wide"), (STORE, 6144, 4096, 4, 256, "narrow"),
    # splits added by the GEMM itself
    (STORE, 3072, 2048, 8, 640, "sum"), (STORE, 6144, 4096, 4, 640, "sum"), (STORE, 4096, 14336, 8, 2048, "sum"),
    (STORE, 4096, 14336, 8, 640, "wide"), (STORE, 1024, 3584, 8, 2048, "sum"), (STORE, 1536, 1024, 4, 2048, "sum"),
])
def test_the_faster_side_is_taken(rules, mode, N, K, splits, M, side):
    assert _side(rules, _args(mode, N, K, M, splits)) == side


@pytest.mark.parametrize("over", [{"x": (1 << 20) + 2}, {"x": (1 << 20) + 8}, {"ldx": 4100}, {"y": (1 << 30) + 4}, {"ldy": 128258},
                                  {"N": 128254}, {"ldx": 1 << 23}])
def test_addresses_and_strides_that_the_wide_tiles_cannot_take(rules, over):
    assert _side(rules, _args(LOGITS, 128256, 4096, 256)) == "wide"
    a = _args(LOGITS, 128256, 4096, 256)
    for k, v in over.items():
        setattr(a, k, v)
    assert not rules["gemm_wide_fits"](a) and _side(rules, a) == "narrow"


def test_segments_that_start_inside_a_tile(rules):
    a = _args(STORE, 6144, 4096, 640, 4, nseg=2)
    a.seg[1].n0 = 4096
    assert _side(rules, a) == "sum"
    a.seg[1].n0 = 4096 + 64
    assert _side(rules, a) == "narrow"
