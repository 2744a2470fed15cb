"""Which kernels a clustering call runs, asked of the library's own rules: the lists of shapes in the GPU
tests name them, and a CPU test holds them to it."""
import ctypes

import paper_2412_03213_amd as ck


class _Dims(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("S", "Hq", "Hkv", "G", "HP")] + [
        ("N_cap", ctypes.c_int64), ("C_cap", ctypes.c_int), ("dtype", ctypes.c_int)]


def _rule(name, restype, *argtypes):
    f = getattr(ck.load_library(), name)
    f.restype, f.argtypes = restype, argtypes
    return f


def assignment(hp, n, C, compute_units=256):
    """'small' (one kernel for all), 'wide', 'stream', 'stream early', or 'few' with the tokens of a chunk,
    and 'one' for a table of one chunk or 'tight' for keys through half of the LDS."""
    i64, i32 = ctypes.c_int64, ctypes.c_int
    if _rule("_ZN2ck17kmeans_small_fitsEli", ctypes.c_bool, i64, i32)(n, C):
        return "small"
    dm = _Dims(1, hp, hp, 1, hp, n, C, ck.CK_BF16)
    tokens = _rule("_ZN2ck18assign_tile_tokensERKNS_4DimsEli", i32, ctypes.POINTER(_Dims), i64, i32)(dm, n, C)
    if tokens == 512:
        if not _rule("_ZN2ck18assign_stream_fitsEi", ctypes.c_bool, i32)(C):
            return "wide"
        return "stream early" if C <= 128 else "stream"
    waves = tokens // 32
    tight = -(-n // tokens) * hp > compute_units * (12 // waves)
    return f"few {tokens}" + (" one" if C <= 64 else " tight" if tight else "")


def update(hp, n, C):
    """'labels', 'chunks' or 'sorted'."""
    i64, i32 = ctypes.c_int64, ctypes.c_int
    dm = _Dims(1, hp, hp, 1, hp, n, C, ck.CK_BF16)
    if _rule("_ZN2ck18update_labels_fitsERKNS_4DimsEli", ctypes.c_bool, ctypes.POINTER(_Dims), i64, i32)(dm, n, C):
        return "labels"
    tokens = _rule("_ZN2ck18assign_tile_tokensERKNS_4DimsEli", i32, ctypes.POINTER(_Dims), i64, i32)(dm, n, C)
    return "chunks" if _rule("_ZN2ck18update_chunks_fitsEil", ctypes.c_bool, i32, i64)(tokens, n) else "sorted"
