"""The rules that choose a kernel by size, called in the built library (they
are host code; no GPU is used): routing in the scoring kernel's shared mode or
in the tile kernel."""

import ctypes

import pytest

from paper_2607_16305_amd import lookme as lk

F32, BF16 = 0, 1
STREAM, SHARED, DTL = 0, 1, 2


class RoutePlan(ctypes.Structure):
    _fields_ = [("mode", ctypes.c_int), ("splits", ctypes.c_int), ("per_split", ctypes.c_int),
                ("part_entries", ctypes.c_int64)]


def route_plan(dt, rows, S, row_bytes, cos=False):
    f = lk.load()._ZN6lookme10route_planEililb
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_bool]
    f.restype = RoutePlan
    return f(dt, rows, S, row_bytes, cos)


@pytest.mark.parametrize("dt,rows,S,row_bytes,mode", [
    # many rows over less than a key tile, or little more than one: the tile
    # kernel took 1.3 to 4 times the shared mode's time
    (BF16, 80000, 64, 128, SHARED), (BF16, 400000, 64, 1024, SHARED),
    (BF16, 131072, 300, 256, SHARED), (BF16, 200000, 300, 512, SHARED),
    (F32, 65536, 64, 2048, SHARED), (F32, 400000, 300, 1024, SHARED),
    (F32, 131072, 300, 2048, SHARED),
    # whole tiles: the tile kernel
    (BF16, 65536, 256, 512, DTL), (BF16, 92160, 1024, 1024, DTL),
    (BF16, 131072, 4096, 128, DTL), (BF16, 400000, 1024, 2048, DTL),
    (F32, 131072, 1024, 512, DTL), (F32, 92160, 4096, 256, DTL),
    # fewer rows than the shared mode's units need
    (BF16, 65408, 64, 128, DTL), (F32, 65408, 300, 256, DTL), (BF16, 4096, 64, 128, DTL),
    # not the tile kernel's: few rows, keys of no whole stages, cosine scores
    (BF16, 4095, 1024, 128, STREAM), (BF16, 65536, 1024, 192, SHARED),
])
def test_routing_mode(dt, rows, S, row_bytes, mode):
    assert route_plan(dt, rows, S, row_bytes).mode == mode
    assert route_plan(dt, rows, S, row_bytes, True).mode != DTL

