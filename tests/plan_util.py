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
