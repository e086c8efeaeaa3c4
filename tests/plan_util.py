"""The library's internal host functions that tests ask for the route of a call, by their C++ names."""
import ctypes

import paper_2506_12024_amd as fq


class _Plan(ctypes.Structure):
    _fields_ = [("mt", ctypes.c_int), ("segments", ctypes.c_int)]


def _fn(name, restype, *argtypes):
    f = getattr(fq.lib, name)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


_i = ctypes.c_int
part_mutex = _fn("_Z13fq_part_mutexii", ctypes.c_void_p, _i, _i)
batch_serves_linear = _fn("_Z22fq_batch_serves_lineariiii", ctypes.c_bool, _i, _i, _i, _i)


class _Desc(ctypes.Structure):  # FqLinearDesc
    _fields_ = ([(n + b, ctypes.c_void_p) for b in "48" for n in ("codes", "scales", "zeros")] + [("w16", ctypes.c_void_p)] +
                [(n + b, ctypes.c_void_p) for b in "23" for n in ("codes", "scales", "zeros")] +
                [("x", ctypes.c_void_p), ("y", ctypes.c_void_p)] + [(n, _i) for n in ("N", "K", "tile_begin", "pad")])


_batch_serves = _fn("_Z15fq_batch_servesPK12FqLinearDescii", ctypes.c_bool, ctypes.c_void_p, _i, _i)


def batch_serves(entries, M):
    """Whether a plan of (N, K, attached widths out of 4, 8, 16) runs on the small-batch kernel (sizes permitting)."""
    table = (_Desc * len(entries))()
    for d, (N, K, widths) in zip(table, entries):
        d.N, d.K = N, K
        d.codes4, d.codes8, d.w16 = (16 if b in widths else None for b in (4, 8, 16))
    return _batch_serves(table, len(entries), M)
