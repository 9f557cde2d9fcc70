"""ctypes view of tests/c_abi/plan_hook.cpp: how the library lays out and cuts the block of approximate cosines and
the reduction of maps, where the text profiles lie, and the order of causal tiles."""
import ctypes as C
import os

_SO = os.path.join(os.path.dirname(os.path.abspath(__file__)), "c_abi", "libplan_hook.so")
SQUARE, WIDE, TALL = 0, 1, 2            # tiles of 128 x 128, 192 x 192, 256 x 192


class GramPlan(C.Structure):
    _fields_ = [("ct", C.c_int64), ("xhat", C.c_int64), ("ttext", C.c_int64), ("cmax", C.c_int64), ("use_gram", C.c_int32), ("splits", C.c_int32),
                ("st_per_split", C.c_int32), ("form", C.c_int32), ("Df", C.c_int32), ("delta", C.c_float)]


class ReducePlan(C.Structure):
    _fields_ = [("total", C.c_int64), ("beyond", C.c_int64), ("row_lanes", C.c_int32), ("strip_groups", C.c_int32), ("rows", C.c_int32),
                ("chunks", C.c_int32), ("combined", C.c_int32)]


def _lib():
    assert os.path.exists(_SO), "tests/c_abi/libplan_hook.so is not built: run `python -m paper_2411_17686_amd.build`"
    return C.CDLL(_SO)


def gram_plan(p):
    g = GramPlan()
    rc = _lib().plan_hook_gram(C.byref(p), C.byref(g))
    assert rc == 0, rc
    return g


def reduce_plan(p, scratch=2 ** 64 - 1):
    r = ReducePlan()
    rc = _lib().plan_hook_reduce(C.byref(p), C.c_uint64(scratch), C.byref(r))
    assert rc == 0, rc
    return r


def causal_tiles(groups, k_tiles, per, full):
    out = (C.c_int32 * (2 * groups * k_tiles))()
    _lib().plan_hook_causal_tiles(groups, k_tiles, per, full, out)
    return list(zip(out[::2], out[1::2]))


def causal_live_first(units, k_tiles):
    return bool(_lib().plan_hook_causal_live_first(units, k_tiles))


def causal_long_first(keys_of_first, keys_of_last):
    return bool(_lib().plan_hook_causal_long_first(keys_of_first, keys_of_last))


def unit_rows_summed(p):
    return bool(_lib().plan_hook_unit_rows_summed(C.byref(p)))
