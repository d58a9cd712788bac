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
                ("lambda_", ctypes.c_float), ("partial", ctypes.c_void_p), ("dev", ctypes.c_void_p), ("parts", ctypes.c_void_p)]


class _GemmPlan(ctypes.Structure):       # GemmF32Plan
    _fields_ = [("three_terms", ctypes.c_bool), ("tile", ctypes.c_int), ("split", ctypes.c_int), ("direct", ctypes.c_bool),
                ("us", ctypes.c_double)]


EPI_STORE, EPI_RMW, EPI_RESID, EPI_SHRINK = range(4)
TILES = ["128x128", "128x64", "64x64", "64x32", "32x32", "16x16"]
X3_TILES = ["128x64", "128x128"]


def forward(lib, B, J, D, have_copy):
    """(mt, ntl, split) of the bf16 forward; mt == 0: the 256 x 256 tiles."""
    f = lib._ZN3sfb16mlr_forward_planElllbb
    f.restype, f.argtypes = _ForwardPlan, [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2
    p = f(B, J, D, have_copy, True)
    return p.mt, p.ntl, p.split


def _plan(lib, kind, B, J, D):
    """The plan that launch_gemm_f32 follows for a contraction of sfb_compute_sf or sfb_apply.

    kind: "logits" and "projections" (X W^T, stored for a row kernel that may add up the k-splits), "shrink" (the same
    operands), "residual" (codes times W) or "apply" (U^T V over B pairs)."""
    f = lib._ZN3sfb13gemm_f32_planERKNS_11GemmF32ArgsE
    f.restype, f.argtypes = _GemmPlan, [ctypes.c_void_p]
    dev = (ctypes.c_int * 64)(CUS, 8)           # DeviceInfo starts with the CU count
    a = _GemmArgs(A=4096, B=4096, partial=4096, dev=ctypes.addressof(dev))
    if kind in ("logits", "projections", "shrink"):
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.epilogue = B, J, D, D, D, J, EPI_SHRINK if kind == "shrink" else EPI_STORE
        if kind == "projections" and J <= 1024 or kind == "logits" and (J <= 1024 or J <= 4096 and B >= CUS):
            a.parts = 4096                      # (dml_scale_adds, mlr_softmax_adds)
    elif kind == "residual":
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.b_kstrided, a.epilogue = B, D, J, J, D, D, True, EPI_RESID
    else:
        a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.a_kstrided, a.b_kstrided, a.epilogue = J, D, B, J, D, D, True, True, EPI_RMW
    return f(ctypes.byref(a))


def gemm_f32(lib, kind, B, J, D):
    """(tile, k split over workgroups, direct loads) where that contraction runs on the fp32 matrix instructions, else None."""
    p = _plan(lib, kind, B, J, D)
    return None if p.three_terms else (TILES[p.tile], p.split, p.direct)


def gemm_f32x3(lib, kind, B, J, D):
    """(tile, k split) where it runs on three bf16 terms per value, else None."""
    p = _plan(lib, kind, B, J, D)
    return (X3_TILES[p.tile], p.split) if p.three_terms else None


def split(lib, kind, B, J, D):
    return _plan(lib, kind, B, J, D).split


def estimate(lib, kind, B, J, D):
    return _plan(lib, kind, B, J, D).us
