"""The dispatch rules of csrc/dispatch.h, compiled by the host compiler."""
import atexit
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
i64 = ctypes.c_int64

MASK_ROUTES = ("quad", "ragged", "turn", "general")


@functools.lru_cache(maxsize=None)
def _rules():
    tmp = tempfile.mkdtemp(prefix="dispatch_rules")
    atexit.register(shutil.rmtree, tmp, True)
    so = os.path.join(tmp, "rules.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "dispatch_probe.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.mask_route_of.argtypes = [i64, i64, ctypes.c_int, i64]
    lib.gemv_takes.argtypes = [i64, i64, i64, ctypes.c_int]
    lib.unmask_words_form_of.argtypes = [i64] * 4
    lib.gather_cols_rows_of.argtypes = [ctypes.c_int] + [i64] * 4
    lib.gather_cols_sparse_of.argtypes = [ctypes.c_int] + [i64] * 4
    lib.gather_rows_single_of.argtypes = [ctypes.c_int, ctypes.c_int] + [i64] * 4
    lib.gemm_plan_of.argtypes = [i64, i64, i64, ctypes.c_int, i64, ctypes.POINTER(i64)]
    lib.launches_of.argtypes = [i64, i64, i64, ctypes.c_void_p]
    return lib


def mask_route(rows, cols, x=None, aligned=False, noise=None, digits=False, cus=256):
    """x: None, "rows", "turned" or "strided"; noise: None, "rows" or "turned"."""
    f = (x is not None) + 2 * (x == "rows") + 4 * (x == "turned") + 8 * aligned + 16 * (noise is not None) + \
        32 * (noise == "turned") + 64 * digits
    return MASK_ROUTES[_rules().mask_route_of(rows, cols, f, cus)]


def gemv(M, N, K, unmask):
    """Whether a product of M rows of A takes the dot-product kernel."""
    return bool(_rules().gemv_takes(M, N, 64 * -(-K // 64), unmask))


def unmask_words(M, N, K, cus=256):
    """(16-row tiles of B, waves) per workgroup."""
    return ((1, 4), (2, 4), (1, 2), (2, 2))[_rules().unmask_words_form_of(M, N, 64 * -(-K // 64), cus)]


def gather_cols(nterms, M, N, cols, cus=256):
    """Rows of d staged per workgroup, 0 if they are read from memory."""
    return _rules().gather_cols_rows_of(nterms, M, N, cols, cus)


def gather_cols_sparse(n, M, N, cols, entries):
    """Whether a column gather of known entries runs its matrices one after the other."""
    return bool(_rules().gather_cols_sparse_of(n, M, N, cols, entries))


def gather_rows_single(n, weight, entries, rows, ncols, cus=256):
    """Whether a row gather over n matrices runs them one after the other."""
    return bool(_rules().gather_rows_single_of(n, weight, entries, rows, ncols, cus))


def gemm_plan(M, N, K, epilogue, cus=256):
    """(form, tiles split, pieces of each) of a tiled product of M > 64 rows;
    epilogue: "store", "accum" or "unmask"."""
    out = (i64 * 3)()
    _rules().gemm_plan_of(M, N, 64 * -(-K // 64), ("store", "accum", "unmask").index(epilogue), cus, out)
    return ("128", "64k", "64")[out[0]], out[1], out[2]


def launches(rows, units, most, stop_after=None):
    """(row0, rows, unit0, units) of each launch of at most ``most`` units."""
    out = []

    def note(*part):
        out.append(part)
        return stop_after is None or len(out) < stop_after

    cb = ctypes.CFUNCTYPE(ctypes.c_int, i64, i64, i64, i64)(note)
    _rules().launches_of(rows, units, most, ctypes.cast(cb, ctypes.c_void_p))
    return out
