"""Which kernel instantiation the library picks for a shape, asked of its own planners (no GPU needed)."""
import ctypes

CUS = 256


class _ForwardPlan(ctypes.Structure):
    _fields_ = [("mt", ctypes.c_int), ("ntl", ctypes.c_int), ("split", ctypes.c_int)]


class _GemmArgs(ctypes.Structure):       # GemmF32Args of csrc/kernels.h
    _fields_ = [("A", ctypes.c_void_p), ("lda", ctypes.c_int64), ("a_kstrided", ctypes.c_bool),
                ("B", ctypes.c_void_p), ("ldb", ctypes.c_int64), ("b_kstrided", ctypes.c_bool),
                ("C", ctypes.c_void_p), ("ldc", ctypes.c_int64),
                ("M", ctypes.c_int64), ("N", ctypes.c_int64), ("K", ctypes.c_int64),
                ("epilogue", ctypes.c_int), ("eta", ctypes.c_float), ("aux", ctypes.c_void_p), ("L_ptr", ctypes.c_void_p),
                ("lambda_", ctypes.c_float), ("partial", ctypes.c_void_p), ("dev", ctypes.c_void_p)]


class _GemmPlan(ctypes.Structure):       # GemmF32Plan
    _fields_ = [("tile", ctypes.c_int), ("split", ctypes.c_int), ("direct", ctypes.c_bool), ("us", ctypes.c_double)]


TILES = ["128x128", "128x64", "64x64", "64x32", "32x32", "16x16"]


def forward(lib, B, J, D, have_copy):
    """(mt, ntl, split) of the bf16 forward; mt == 0: the 256 x 256 tiles."""
    f = lib._ZN3sfb16mlr_forward_planElllbb
    f.restype, f.argtypes = _ForwardPlan, [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2
    p = f(B, J, D, have_copy, True)
    return p.mt, p.ntl, p.split


def gemm_f32(lib, kind, B, J, D):
    """(tile, k split over workgroups, direct loads) of an fp32 contraction of sfb_compute_sf or sfb_apply.

    kind: "logits" (also the projections and the shrink step: X W^T), "residual" (codes times W) or "apply"
    (U^T V over B pairs)."""
    f = lib._ZN3sfb13gemm_f32_planERKNS_11GemmF32ArgsE
    f.restype, f.argtypes = _GemmPlan, [ctypes.c_void_p]
    dev = (ctypes.c_int * 64)(CUS, 8)           # DeviceInfo starts with the CU count
    a = _GemmArgs(A=4096, B=4096, partial=4096, dev=ctypes.addressof(dev))
    if kind == "logits":
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc = B, J, D, D, D, J
    elif kind == "residual":
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.b_kstrided = B, D, J, J, D, D, True
    else:
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.a_kstrided, a.b_kstrided = J, D, B, J, D, D, True, True
    p = f(ctypes.byref(a))
    return TILES[p.tile], p.split, p.direct


class _X3Plan(ctypes.Structure):         # GemmF32x3Plan of csrc/gemm_f32.h
    _fields_ = [("tile", ctypes.c_int), ("split", ctypes.c_int), ("us", ctypes.c_double)]


X3_TILES = ["128x64", "128x128"]


def gemm_f32x3(lib, kind, B, J, D, max_split=8):
    """(tile, k split) where the kernel on three bf16 terms takes that contraction, else None."""
    f = lib._ZN3sfb15gemm_f32x3_planERKNS_11GemmF32ArgsEi
    f.restype, f.argtypes = _X3Plan, [ctypes.c_void_p, ctypes.c_int]
    g = lib._ZN3sfb13gemm_f32_planERKNS_11GemmF32ArgsE
    g.restype, g.argtypes = _GemmPlan, [ctypes.c_void_p]
    dev = (ctypes.c_int * 64)(CUS, 8)
    a = _GemmArgs(A=4096, B=4096, partial=4096, dev=ctypes.addressof(dev))
    if kind == "logits":
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc = B, J, D, D, D, J
    elif kind == "residual":
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.b_kstrided, a.epilogue = B, D, J, J, D, D, True, 2
    else:
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.a_kstrided, a.b_kstrided, a.epilogue = J, D, B, J, D, D, True, True, 1
    p = f(ctypes.byref(a), max_split)
    return (X3_TILES[p.tile], p.split) if p.tile >= 0 and p.us < g(ctypes.byref(a)).us else None
