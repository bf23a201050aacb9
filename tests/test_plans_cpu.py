"""The rules that choose a kernel by size, called in the built library (they
are host code; no GPU is used): routing in the scoring kernel's shared mode or
in the tile kernel, the partials that its splits need, the products and the
projections that run on 256 x 256 tiles, and the ranges of the relevance MLP's
second layer."""

import ctypes

import pytest

from paper_2607_16305_amd import lookme as lk

F32, BF16 = 0, 1
STREAM, SHARED, DTL = 0, 1, 2
FAKE = 0x7F0000100000          # 256-byte aligned stand-in address, never dereferenced


class RoutePlan(ctypes.Structure):
    _fields_ = [("mode", ctypes.c_int), ("splits", ctypes.c_int), ("per_split", ctypes.c_int),
                ("part_entries", ctypes.c_int64)]


def route_plan(dt, rows, S, row_bytes, cos=False):
    f = lk.load()._ZN6lookme10route_planEililb
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_bool]
    f.restype = RoutePlan
    return f(dt, rows, S, row_bytes, cos)


def product_phased(dt, rows, cols, k_bytes, batches=1, tile_cols=256):
    f = lk.load()._ZN6lookme14product_phasedEillill
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64,
                  ctypes.c_int64]
    f.restype = ctypes.c_bool
    return f(dt, rows, cols, tile_cols, batches, k_bytes)


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


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("S", [1, 300, 1024, 4096, 8448, 16384])
def test_routing_plans_fit_their_limits(dt, S):
    """Every key tile is in one range, a range holds at most 16 tiles, split
    blocks have a counter each, and but for the first split that holds the
    bias table a plan makes at most 2048 units."""
    tiles = -(-S // 256)
    first = 1
    while -(-tiles // first) > 16:
        first *= 2
    for rows in list(range(4096, 70000, 1111)) + list(range(70000, 1200000, 31013)):
        for rb in (128, 512, 2048):
            p = route_plan(dt, rows, S, rb)
            if p.mode != DTL:
                continue
            blocks = -(-rows // 128)
            assert p.per_split <= 16 and (p.splits - 1) * p.per_split < tiles
            assert p.splits * p.per_split >= tiles
            assert p.part_entries == (blocks * p.splits * 128 if p.splits > 1 else 0)
            if p.splits > 1:
                assert blocks <= 4096
                assert p.splits <= first or blocks * p.splits <= 2048, (rows, rb)


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("S", [16, 300, 1024, 4096, 8448, 16384])
@pytest.mark.parametrize("key_bytes", [64, 256, 1024])
@pytest.mark.parametrize("score", [lk.LOOKME_SCORE_DOT, lk.LOOKME_SCORE_COS])
def test_a_workspace_serves_every_smaller_batch(dt, S, key_bytes, score):
    """lookme_workspace_size never falls with the batch, and holds what the
    plan of the batch itself writes."""
    desc = lk.lookme_desc_t(S, 8, key_bytes // (4 if dt == F32 else 2), 64, 4, dt, score)
    h = lk.lookme_create(desc, FAKE, FAKE, FAKE)
    try:
        last = 0
        for n in list(range(1, 300, 7)) + list(range(300, 20000, 97)) + \
                list(range(20000, 800000, 640)):
            size = lk.lookme_workspace_size(h, 1, n)
            assert size >= last, n
            last = size
            p = route_plan(dt, n, S, key_bytes, score == lk.LOOKME_SCORE_COS)
            assert p.part_entries * 8 < size, n
        for layers, n in ((4, 12288), (4, 12416), (3, 16555), (2, 24801)):
            assert lk.lookme_workspace_size(h, layers, n) <= \
                lk.lookme_workspace_size(h, layers, n + 1000)
            assert lk.lookme_workspace_size(h, layers - 1, n) <= \
                lk.lookme_workspace_size(h, layers, n)
    finally:
        lk.lookme_destroy(h)


@pytest.mark.parametrize("dt,tiles,k_bytes,phased", [
    (BF16, 47, 4096, False), (BF16, 48, 4096, True), (BF16, 128, 1024, False),
    (BF16, 129, 1024, True),
    # float32: where the rounds, of whole tiles or of quarters, are nearly full
    (F32, 48, 8192, False), (F32, 50, 8192, True), (F32, 64, 8192, True), (F32, 90, 8192, False),
    (F32, 128, 8192, True), (F32, 190, 8192, False), (F32, 225, 8192, True),
    (F32, 256, 2048, True), (F32, 300, 8192, True), (F32, 385, 8192, False),
    (F32, 450, 8192, True), (F32, 512, 4096, True), (F32, 5000, 4096, True),
])
def test_products_on_large_tiles(dt, tiles, k_bytes, phased):
    assert product_phased(dt, 256 * tiles, 256, k_bytes) == phased
    assert product_phased(dt, 256, 256, k_bytes, batches=tiles) == phased
    assert product_phased(dt, 256, 128 * tiles, k_bytes, tile_cols=128) == phased


@pytest.mark.parametrize("dt,rows,cols,k_bytes,batches,tile_cols", [
    # one column tile, a quarter or half of it padding: two to three times the
    # time of 64 x 64 tiles
    (F32, 131072, 64, 4096, 1, 256), (F32, 131072, 128, 4096, 1, 256),
    (BF16, 33000, 64, 4096, 1, 256), (BF16, 16385, 128, 8192, 1, 256),
    # a row block of 1 or 44 rows in each of four layers
    (F32, 257, 4096, 8192, 4, 128), (F32, 300, 4096, 8192, 4, 128),
    (BF16, 300, 1600, 2304, 4, 128), (BF16, 600, 1600, 2304, 2, 128),
    # both edges, short sums
    (BF16, 12000, 640, 256, 1, 256), (BF16, 16385, 384, 1024, 1, 256),
])
def test_products_mostly_of_padding_on_small_tiles(dt, rows, cols, k_bytes, batches, tile_cols):
    assert not product_phased(dt, rows, cols, k_bytes, batches, tile_cols)


@pytest.mark.parametrize("dt,n,cols,k_bytes,one_round", [
    (BF16, 32768, 512, 8192, True), (BF16, 8192, 2048, 1024, True), (BF16, 16384, 512, 1024, True),
    (BF16, 23040, 512, 1024, True), (F32, 16384, 896, 8192, True), (F32, 8192, 2048, 512, True),
    # fewer tiles, or more than a round of them
    (BF16, 23040, 512, 4096, False), (F32, 23040, 512, 4096, False),
    (BF16, 33000, 512, 4096, False), (BF16, 16128, 512, 1024, False),
    # mostly padding: 64 x 64 tiles take a third to nine tenths of the time
    (F32, 65536, 64, 8192, False), (F32, 65536, 192, 8192, False), (F32, 32768, 320, 4096, False),
    (BF16, 32768, 64, 1024, False), (BF16, 65536, 64, 8192, False), (BF16, 16384, 320, 1024, False),
    (BF16, 8192, 896, 1024, False),
    # no whole K stages
    (BF16, 32768, 512, 8256, False),
])
def test_projections_of_one_round(dt, n, cols, k_bytes, one_round):
    f = lk.load()._ZN6lookme17project_one_roundEilll
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64]
    f.restype = ctypes.c_bool
    assert f(dt, n, cols, k_bytes) == one_round


def relevance_ranges(rows, P, k):
    f = lk.load()._ZN6lookme18relevance_ranges32Elii
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    f.restype = ctypes.c_int
    return f(rows, P, k)


@pytest.mark.parametrize("rows,P,k,ranges", [
    # two workgroups a CU also where one a CU is whole (with one the Zipf
    # batch's lookup took 395 us against 329)
    (32768, 4096, 16, 2), (32768, 1024, 8, 2), (16384, 4096, 16, 4), (16384, 2048, 8, 4),
    (8192, 4096, 16, 8), (4096, 4096, 16, 16),
    (32769, 4096, 16, 1), (16385, 4096, 16, 2), (20011, 1000, 8, 2), (12000, 1024, 16, 4),
    # ranges too short for the second one
    (16384, 512, 16, 2), (32768, 512, 16, 1), (28000, 256, 8, 1), (8192, 1024, 16, 4),
    # as many as a range's b2 needs
    (65536, 4097, 8, 2), (65536, 65536, 8, 16), (65536, 65537, 8, 0),
])
def test_relevance_ranges(rows, P, k, ranges):
    assert relevance_ranges(rows, P, k) == ranges


def test_relevance_ranges_hold_their_lists():
    """A split's lists, k entries of 8 bytes a range and row, fit the logits'
    4 P bytes a row that hold them (the launcher refuses others), and no
    range is shorter than its k."""
    for rows in (4096, 4097, 6000, 8192, 16384, 20011, 32768, 32769, 65536):
        for P in (1, 16, 127, 128, 255, 256, 257, 511, 1000, 1024, 4095, 4096, 5000, 65536):
            for k in (1, 4, 7, 8, 16):
                s = relevance_ranges(rows, P, k)
                assert s >= 1
                assert s == 1 or (s * k * 2 <= P and P // s >= max(k, 128))
                assert s == 1 or (rows + 127) // 128 * s <= 512 or -(-P // (s // 2)) > 4096
