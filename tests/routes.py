"""The library's own rules of dispatch (csrc/wht_route.h, built for the host as csrc/route_query.cpp), so that a test that says
which kernel it runs asks for sizes instead of restating limits."""
import ctypes
import functools

from paper_2603_08343_amd import build

WAYS = ("plain", "through", "pair", "stream", "flow")        # Way, in its order
ONE_PASS, PERSISTENT = WAYS[:3], WAYS[3:]
OUTS = ("y", "resid", "stats")                               # Out


@functools.lru_cache(maxsize=None)
def _lib():
    lib = ctypes.CDLL(build.ROUTE_LIB)
    i32, i64 = ctypes.c_int32, ctypes.c_int64
    lib.wht_query_forward_steps.argtypes = [i32, i32, i32, i32, ctypes.POINTER(ctypes.c_double), ctypes.POINTER(i32)]
    lib.wht_query_forward.argtypes = [i32, i32, i32, i32, i64]
    lib.wht_query_dx_through.argtypes = [i32, i32, i32, i64]
    lib.wht_query_sums_store.argtypes = [i32, i32, i32]
    lib.wht_query_few_elements.argtypes = [i32, i32]
    lib.wht_query_few_elements.restype = i64
    return lib


def _code(dtype):
    return {"f32": 0, "bf16": 1}[dtype]


def row_bytes(dtype, d):
    return d * (4 if dtype == "f32" else 2)


def tokens(dtype, d, mib):
    """The first token count whose tensor has this many MiB."""
    return max(1, -(-int(mib * (1 << 20)) // row_bytes(dtype, d)))


def steps(dtype, d, out="y", butterfly=False):
    """[(MiB from which on, way)], from 0 on."""
    mib, way = (ctypes.c_double * 8)(), (ctypes.c_int32 * 8)()
    n = _lib().wht_query_forward_steps(_code(dtype), d, int(butterfly), OUTS.index(out), mib, way)
    assert n > 0, (dtype, d, out)
    return [(mib[i], WAYS[way[i]]) for i in range(n)]


def way(dtype, d, N, out="y", butterfly=False):
    w = _lib().wht_query_forward(_code(dtype), d, int(butterfly), OUTS.index(out), N)
    assert w >= 0, (dtype, d, N, out)
    return WAYS[w]


def persistent_from(dtype, d, out="y", butterfly=False):
    """The first token count from which on every call is the persistent kernel's."""
    s = steps(dtype, d, out, butterfly)
    last = max(i for i, (_, w) in enumerate(s) if w in ONE_PASS)
    return tokens(dtype, d, s[last + 1][0])


def dx_through(dtype, d, N, grads=True):
    return bool(_lib().wht_query_dx_through(_code(dtype), d, int(grads), N))


def sums_store(dtype, d, dx=True):
    """How the partial rows of dalpha and dbeta are written."""
    return ("plain", "stream", "through")[_lib().wht_query_sums_store(_code(dtype), d, int(dx))]


def few_elements(dtype, d):
    return _lib().wht_query_few_elements(_code(dtype), d)
