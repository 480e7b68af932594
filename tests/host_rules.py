"""The library's rules on sizes (csrc/fcp_sizes.h, plain C++), compiled by themselves for the tests."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "host_rules.so")
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2602_21788_amd", "csrc"),
                               "-o", so, os.path.join(ROOT, "tests", "host_rules.cpp")])
        L = ctypes.CDLL(so)
    i32, i64, P = ctypes.c_int32, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)
    L.forward_plan.argtypes = [i32, i32, i32, i32, i32, i64, i32, i32, i64, P]
    L.forward_plan.restype = None
    for f in (L.static_bytes, L.scratch_area_bytes):
        f.argtypes, f.restype = [i32, i32, i64, i32], i64
    L.persistent_blocks.argtypes, L.persistent_blocks.restype = [i64, i64], i64
    L.first_unit.argtypes, L.first_unit.restype = [i32, i32, i32, i32, P], None
    L.head_queues.argtypes, L.head_queues.restype = [i32, i32], i32
    L.unit_numbers.argtypes, L.unit_numbers.restype = [i32, i32, i32, P], None
    L.bwd_kv_cap.argtypes, L.bwd_kv_cap.restype = [i32, i64], i64
    L.bwd_q_cap.argtypes, L.bwd_q_cap.restype = [i32, i32, i64], i64
    L.forward_alone.argtypes, L.forward_alone.restype = [i32, i32, i64, i32, i64, i32], i32
    L.delta_streams_do.argtypes, L.delta_streams_do.restype = [i32, i32, i32], i32
    L.alone_order.argtypes, L.alone_order.restype = [i32, i64, i64, i32], i32
    L.deals_first.argtypes, L.deals_first.restype = [i32, i32, i32, i32], i32
    L.keeps_reserve.argtypes, L.keeps_reserve.restype = [i32, i32], i32
    L.backward_way.argtypes, L.backward_way.restype = [i32, i32, i32, i32, i32, i64, i32], i32
    return L


def forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, area, n_cu=256):
    """(tile rows, two heads per unit, tiles the list has room for, bytes of its region)."""
    out = (ctypes.c_int64 * 4)()
    lib().forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, n_cu, area, out)
    return tuple(out)


def persistent_blocks(resident, units):
    return lib().persistent_blocks(resident, units)


def first_unit(place, places, key_units, n_long):
    """(key units dealt, the block's first key unit, its first row unit); -1: none of that list."""
    out = (ctypes.c_int64 * 3)()
    lib().first_unit(place, places, key_units, n_long, out)
    return tuple(out)


def head_queues(per_tile, in_turn):
    return lib().head_queues(per_tile, in_turn)


def unit_numbers(block, queues, in_turn):
    """(counter, mul, add): number i of the counter is unit mul i + add of the queue's heads."""
    out = (ctypes.c_int64 * 3)()
    lib().unit_numbers(block, queues, in_turn, out)
    return tuple(out)


def deals_first(units, blocks, per_block, longest):
    return bool(lib().deals_first(units, blocks, per_block, longest))


def keeps_reserve(dealt, longest):
    return bool(lib().keeps_reserve(dealt, longest))


def backward_caps(tq, tkv, n_work):
    """Tiles that the key-tile and the query-tile list have room for."""
    return lib().bwd_kv_cap(tkv, n_work), lib().bwd_q_cap(tq, tkv, n_work)


ONE_PASS, MANY_SHORT, EITHER = 1, 2, 4


def backward_way(hq, hkv, head_dim, tq, tkv, n_work, n_cu=256):
    return lib().backward_way(hq, hkv, head_dim, tq, tkv, n_work, n_cu)
