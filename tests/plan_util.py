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


def batch_serves(entries, M, own_x=False):
    """Whether a plan of (N, K, attached widths) runs on the small-batch kernel (sizes permitting); own_x: each entry has an x of its own."""
    table = (_Desc * len(entries))()
    for i, (d, (N, K, widths)) in enumerate(zip(table, entries)):
        d.N, d.K, d.x = N, K, 16 + 16 * (i if own_x else 0)
        d.codes2, d.codes3, d.codes4, d.codes8, d.w16 = (16 if b in widths else None for b in (2, 3, 4, 8, 16))
    return _batch_serves(table, len(entries), M)


batch_serves_narrow = _fn("_Z22fq_batch_serves_narrowiiii", ctypes.c_bool, _i, _i, _i, _i)  # a single call at 2 or 3 bits
batch_serves_slab = _fn("_Z20fq_batch_serves_slabiii", ctypes.c_bool, _i, _i, _i)  # a slab of a 3-bit prompt


_prompt_plan = _fn("_Z14fq_prompt_planiiiii", _Plan, _i, _i, _i, _i, _i)
_w8a8_plan = _fn("_Z19fq_w8a8_prompt_planiiibii", _Plan, _i, _i, _i, ctypes.c_bool, _i, _i)


def prompt_plan(M, N, K, bits, cus=256):
    """(blocks of 32 tokens of a tile, segments of K) of fq_linear's GEMM; (0, 0): the 256 x 256 tiles."""
    p = _prompt_plan(N, K, bits, M, cus)
    return p.mt, p.segments


def w8a8_large_blocks(M, N, cus=256):
    """Blocks of 64 tokens of the large W8A8 tiles for groups of 128 (the launcher's rule)."""
    t3, t2 = ((M + bm - 1) // bm * ((N + 255) // 256) for bm in (192, 128))
    return 2 if (t2 + cus - 1) // cus * 2 * 8 < (t3 + cus - 1) // cus * 3 * 7 else 3


def w8a8_plan(M, N, K, per_row, cus=256):
    """(blocks of 64 tokens of a tile, segments of K) of fq_linear_w8a8; (0, 0): the large tiles."""
    p = _w8a8_plan(N, K, M, per_row, w8a8_large_blocks(M, N, cus), cus)
    return p.mt, p.segments

_part_bank = _fn("_Z12fq_part_bankP12ihipStream_tPi", _i, ctypes.c_void_p, ctypes.c_void_p)


def part_bank(stream):
    """The index of a stream's array for partial sums on the current device, -1 if it has none."""
    return _part_bank(stream, ctypes.byref(_i()))


stream_bank = _fn("_Z14fq_stream_bankP12ihipStream_t", _i, ctypes.c_void_p)  # -1: no copy of the static scratch for this stream


class _Entropy(ctypes.Structure):
    _fields_ = [("threads", ctypes.c_int), ("pieces", ctypes.c_int), ("fine", ctypes.c_int)]


_entropy_route = _fn("_Z16fq_entropy_routeiibbbi", _Entropy, _i, _i, ctypes.c_bool, ctypes.c_bool, ctypes.c_bool, _i)


def entropy_route(R, V, kl, half, vec, cus=256):
    """(threads, pieces of a row, S and Sb in double) of an entropy call."""
    r = _entropy_route(R, V, kl, half, vec, cus)
    return r.threads, r.pieces, r.fine
