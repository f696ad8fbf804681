"""The library's internal GEMM launches (kernels.h) called from tests: the C++
functions by their mangled names, and their argument blocks."""
import ctypes

from paper_2402_15758_amd import binding as B

EPI_F32, EPI_SILU, EPI_SWIGLU, EPI_QKV, EPI_PARTIAL, EPI_ZIN = 0, 2, 3, 4, 5, 6


class StreamPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("row_tiles", "row_blocks", "runs", "run", "long_runs", "mapped")]


class GemmEpi(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_int), ("out_f", ctypes.c_void_p), ("ldo", ctypes.c_int),
                ("out_t", ctypes.c_void_p), ("o_mtiles", ctypes.c_int), ("part", ctypes.c_void_p),
                ("pos", ctypes.c_void_p), ("kvoff", ctypes.c_void_p), ("qrow", ctypes.c_void_p),
                ("kbase", ctypes.c_void_p), ("vbase", ctypes.c_void_p), ("head_stride", ctypes.c_int64),
                ("qout", ctypes.c_void_p), ("ldq", ctypes.c_int), ("rcos", ctypes.c_void_p),
                ("rsin", ctypes.c_void_p), ("H", ctypes.c_int), ("hd", ctypes.c_int)]


class GemmShape(ctypes.Structure):
    _fields_ = [("skip", ctypes.c_void_p), ("X", ctypes.c_void_p), ("x_mtiles", ctypes.c_int), ("M", ctypes.c_int),
                ("W", ctypes.c_void_p), ("N", ctypes.c_int), ("K", ctypes.c_int), ("nb_off", ctypes.c_int),
                ("nb_count", ctypes.c_int), ("splits", ctypes.c_int)]


def fn(name, restype):
    f = B.lib()[name]
    f.restype = restype
    return f


def mcap(M):
    return next((c for c in (16, 32, 64) if M <= c), -(-M // 128) * 128)


def stream_plan(M, nbc, splits):
    return fn("_Z16gemm_stream_planiiii", StreamPlan)(M, nbc, splits, mcap(M) // 16)


def splits_of(bf16, cols, K):
    return fn("_Z16gemm_pick_splitsiii", ctypes.c_int)(cols, K, bf16)


def rows_takes(bf16, M, cols, K, kind):
    return fn("_Z15gemm_rows_takesiiiiii", ctypes.c_bool)(bf16, M, cols // 16, K, splits_of(bf16, cols, K), kind)


def wide_takes(bf16, M, cols, K):
    return fn("_Z15gemm_wide_takesiiiiii", ctypes.c_bool)(bf16, M, cols // 16, K, splits_of(bf16, cols, K),
                                                          mcap(M) // 16)


def wide_tile(M, cols, K):
    s = splits_of(1, cols, K)
    return fn("_Z14gemm_wide_tileiiii", ctypes.c_int)(M, cols // 16, K // 32 // s, s)


def partials(bf16, M, cols, K, kind, mtiles):
    return fn("_Z13gemm_partialsiiiiii", ctypes.c_int)(bf16, M, cols, K, mtiles, kind)


def partial_rows(bf16, max_M, cols, K, kind):
    return fn("_Z17gemm_partial_rowsiiiii", ctypes.c_int64)(bf16, max_M, cols, K, kind)


def wide_sums_slices(M, cols, kind):
    return fn("_Z21gemm_wide_sums_slicesiii", ctypes.c_bool)(M, cols // 16, kind)


def _launch(f, lead, shape, epi, stream):
    f.argtypes = [ctypes.c_int] * len(lead) + [ctypes.c_void_p] * 5
    return f(*lead, ctypes.addressof(shape), ctypes.addressof(epi), stream, None, None)


def launch(bf16, shape, epi, stream):
    return _launch(fn("_Z11launch_gemmiRK9GemmShapeRK7GemmEpiP12ihipStream_tP11ihipEvent_tS8_", ctypes.c_bool), (bf16,),
                   shape, epi, stream)


def launch_wide(shape, epi, stream):
    _launch(fn("_Z16launch_gemm_wideRK9GemmShapeRK7GemmEpiP12ihipStream_tP11ihipEvent_tS8_", None), (), shape, epi,
            stream)
