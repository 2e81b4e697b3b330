"""The library's own choice of kernels, read from its internal (C++) planning functions; host code only."""
import ctypes as C

import paper_2602_01027_amd as S


class _PrefillWorkspace(C.Structure):
    _fields_ = [("xperm_bytes", C.c_int64), ("ytmp_bytes", C.c_int64)]


class DecodePlan(C.Structure):
    _fields_ = [("gemv", C.c_bool), ("grid", C.c_int32), ("lds_bytes", C.c_int32), ("slots", C.c_int32), ("max_slabs", C.c_int32),
                ("mb", C.c_int32), ("nw", C.c_int32), ("acc", C.c_int32), ("resident", C.c_bool), ("ra", C.c_int32),
                ("rs", C.c_int32), ("workspace_bytes", C.c_int64)]


def _call(symbol, result, *args):
    f = getattr(S.load_library(), symbol)
    f.restype, f.argtypes = result, [C.c_int32] * len(args)
    return f(*args)


def chunked(N, K, M):
    """Do 17 <= M <= 128 rows run as chunks of 16 through the decode kernels?"""
    return _call("_ZN4sfmp18use_chunked_decodeEiii", C.c_bool, N, K, M)


def prefill_bytes(N, K, M):
    """(staged activations, product or partial products) of a matrix-core call's workspace."""
    p = _call("_ZN4sfmp17prefill_workspaceEiii", _PrefillWorkspace, N, K, M)
    return p.xperm_bytes, p.ytmp_bytes


def decode_plan(N, K, M, group=128):
    return _call("_ZN4sfmp16make_decode_planEiiiib", DecodePlan, N, K, M, group, False)


class _GemmArgs(C.Structure):
    _fields_ = [("X", C.c_void_p), ("M", C.c_int32), ("col_perm", C.c_void_p), ("L", C.POINTER(S.SfmpLayout))] + [
        (n, C.c_void_p) for n in ("s2", "s3", "s4", "index", "scales", "zeros", "bitmap", "row_perm", "Y", "workspace")] + [
        ("workspace_bytes", C.c_int64)]


class SmallBatchConfig(C.Structure):
    _fields_ = [("mb", C.c_int32), ("nw", C.c_int32), ("slots", C.c_int32), ("acc", C.c_int32), ("resident", C.c_bool),
                ("rs", C.c_int32), ("ra", C.c_int32)]


def _gemm_args(layouts, M, X=None, Y=None):
    """Arguments of products of M rows; X, Y: device addresses (never dereferenced here)."""
    args = (_GemmArgs * len(layouts))()
    for i, layout in enumerate(layouts):
        args[i].M, args[i].L = M, C.pointer(layout)
        args[i].X, args[i].Y = X[i] if X else None, Y[i] if Y else None
    return args


def batched_config(layouts, M, X=None, Y=None):
    """(configuration, workgroups per problem) of one small-batch launch of several matrices."""
    n = len(layouts)
    args = _gemm_args(layouts, M, X, Y)
    g, c, g64 = (C.c_int32 * 8)(), SmallBatchConfig(), C.c_bool()
    f = S.load_library()._ZN4sfmp12batch_configEPK8GemmArgsiiPiPNS_13RSkinnyConfigEPb
    f.restype = C.c_int
    assert f(args, C.c_int(n), C.c_int32(M), g, C.byref(c), C.byref(g64)) == 0
    return c, list(g[:n])


class _PrefillForm(C.Structure):
    _fields_ = [("mi", C.c_int32), ("kg", C.c_int32), ("ksplit", C.c_int32)]


def launched_form(N, K, M):
    """(16-row blocks of a wavefront, K groups of a workgroup, K ranges) of a matrix-core call; (0, 1, 1): prefill_kernel."""
    f = _call("_ZN4sfmp19choose_prefill_formEiii", _PrefillForm, N, K, M)
    return f.mi, f.kg, f.ksplit


def chunks_without_staging(N, K, M, group=128):
    """Do 17 <= M <= 128 rows beyond the documented chunked shapes run in chunks, without touching the workspace?"""
    return _call("_ZN4sfmp26use_chunks_without_stagingEiiii", C.c_bool, N, K, M, group)


def launched_decode_plan(layout, M, X, Y):
    """The plan of a single small-batch launch with these activations and this output."""
    f = S.load_library()._ZN4sfmp14decode_plan_ofERK8GemmArgs
    f.restype = DecodePlan
    return f(_gemm_args([layout], M, [X], [Y]))


def runs_in_chunks(layout, M, X, Y):
    """Do 17 <= M <= 128 rows run in chunks with these activations and this output?"""
    f = S.load_library()._ZN4sfmp14runs_in_chunksERK8GemmArgs
    f.restype = C.c_bool
    return f(_gemm_args([layout], M, [X], [Y]))


class _PrefillTail(C.Structure):
    _fields_ = [("mi", C.c_int32), ("tile_rows", C.c_int32)]


def launched_tail(N, K, M):
    """(16-row blocks of a wavefront, tile rows) of the tail of a matrix-core call in two forms; (0, 0): one form."""
    t = _call("_ZN4sfmp19choose_prefill_tailEiii", _PrefillTail, N, K, M)
    return t.mi, t.tile_rows


def stores_past_caches(N, M):
    """Does the un-permute pass of a matrix-core call store its result past the caches?"""
    return _call("_ZN4sfmp18stores_past_cachesEii", C.c_bool, N, M)


def scatter_threads(N, M):
    """Threads of a workgroup (one row) of that pass."""
    return _call("_ZN4sfmp15scatter_threadsEii", C.c_int32, N, M)
