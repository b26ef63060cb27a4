"""Host functions of the library that are not part of its C interface (GEMM dispatch and launches), for tests of the kernels behind it."""
import ctypes as C

from paper_2601_13155_amd import binding

EPI_STORE, EPI_SILU_MUL, EPI_RESIDUAL, EPI_SUMSQ, EPI_ROPE, EPI_ROPE_STORE, EPI_SILU_MUL_T = range(7)


class GemmArgs(C.Structure):
    """spts::GemmArgs of csrc/spts_internal.h, field by field."""
    _fields_ = [("A", C.c_void_p), ("lda", C.c_int64), ("a_idx", C.c_void_p), ("a_rows", C.c_int64), ("A1", C.c_void_p),
                ("B0", C.c_void_p), ("B1", C.c_void_p), ("ldb", C.c_int64), ("C", C.c_void_p), ("ldc", C.c_int64), ("c_idx", C.c_void_p),
                ("Ct", C.c_void_p), ("ldct", C.c_int64), ("part", C.c_void_p), ("part_ld", C.c_int32), ("rope", C.c_void_p),
                ("head_dim", C.c_int32), ("rope_idx", C.c_void_p), ("rope_scale", C.c_float), ("n_split", C.c_int32), ("C2", C.c_void_p),
                ("ldc2", C.c_int64), ("b_rows1", C.c_int64), ("M", C.c_int64), ("N", C.c_int32), ("K", C.c_int32), ("epi", C.c_int32),
                ("c_is_f32", C.c_int32), ("ksplit", C.c_int32), ("nfull", C.c_int32), ("part32", C.c_void_p), ("a_slab", C.c_int32),
                ("b_slab", C.c_int32), ("b_rows", C.c_int64), ("c_slab", C.c_int32)]


class SmallPlan(C.Structure):
    _fields_ = [("tm", C.c_int), ("ksplit", C.c_int)]


def _fn(mangled, res, *args):
    f = getattr(binding.load(), mangled)
    f.restype, f.argtypes = res, args
    return f


_ARGS = C.POINTER(GemmArgs)


def tile32_supported(a, bf16):
    return _fn("_ZN4spts21gemm_tile32_supportedERKNS_8GemmArgsEb", C.c_bool, _ARGS, C.c_bool)(a, bf16)


def mfma_supported(a):
    return _fn("_ZN4spts19gemm_mfma_supportedERKNS_8GemmArgsE", C.c_bool, _ARGS)(a)


def launch_generic(a, bf16, stream=None):
    return _fn("_ZN4spts19launch_gemm_genericERKNS_8GemmArgsEbP12ihipStream_t", C.c_int, _ARGS, C.c_bool, C.c_void_p)(a, bf16, stream)


def pick_split(M, N, K, epi):
    """(ksplit, nfull) of the 256-wide kernel's plan."""
    nfull = C.c_int32(0)
    ks = _fn("_ZN4spts15gemm_pick_splitEliiiPi", C.c_int, C.c_int64, C.c_int32, C.c_int32, C.c_int, C.POINTER(C.c_int32))(M, N, K, epi, nfull)
    return ks, nfull.value


def small_pick(a, part_bytes):
    """(tm, ksplit) of the short-product kernel where the dispatch prefers it to the 256-wide one, else None."""
    ks, nfull = pick_split(a.M, a.N, a.K, a.epi)
    plan = SmallPlan()
    f = _fn("_ZN4spts15gemm_small_pickERKNS_8GemmArgsEiimPNS_13GemmSmallPlanE", C.c_bool, _ARGS, C.c_int, C.c_int, C.c_size_t, C.POINTER(SmallPlan))
    return (plan.tm, plan.ksplit) if f(a, ks, nfull, part_bytes, plan) else None


def small_part_bytes(a, tm, ksplit):
    return _fn("_ZN4spts21gemm_small_part_bytesERKNS_8GemmArgsERKNS_13GemmSmallPlanE", C.c_size_t, _ARGS, C.POINTER(SmallPlan))(a, SmallPlan(tm, ksplit))


def small_supported(a):
    return _fn("_ZN4spts20gemm_small_supportedERKNS_8GemmArgsE", C.c_bool, _ARGS)(a)


def launch_small(a, tm, ksplit, stream):
    return _fn("_ZN4spts17launch_gemm_smallERKNS_8GemmArgsERKNS_13GemmSmallPlanEP12ihipStream_t", C.c_int, _ARGS, C.POINTER(SmallPlan),
               C.c_void_p)(a, SmallPlan(tm, ksplit), stream)


def launch_wide(a, stream):
    return _fn("_ZN4spts16launch_gemm_mfmaERKNS_8GemmArgsEP12ihipStream_t", C.c_int, _ARGS, C.c_void_p)(a, stream)


def topk_mean(vals, ld, rows, n, k, out, bf16, stream):
    return _fn("_ZN4spts16launch_topk_meanEPKvllllPfbP12ihipStream_t", C.c_int, C.c_void_p, C.c_int64, C.c_int64, C.c_int64, C.c_int64, C.c_void_p, C.c_bool,
               C.c_void_p)(vals, ld, rows, n, k, out, bf16, stream)
