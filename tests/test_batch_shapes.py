"""The built-in tile shapes of a mixed-order batch (those of a plan without
autotuning and of the static call, which share one selection), on the host: the
shapes on both sides of every line of the rule, and that a call whose tiles
can fit the static call's table gets shapes that do."""
import ctypes
import os

import pytest

MAX_TILES = 32768
F64, F32 = 0, 1
FULL, ALIAS = 0, 1      # the library's internal layout codes


class Order(ctypes.Structure):
    _fields_ = [("nq", ctypes.c_int), ("elements", ctypes.c_int64)]


class Tile(ctypes.Structure):
    _fields_ = [("epb", ctypes.c_int), ("lay", ctypes.c_int)]


@pytest.fixture(scope="module")
def shapes():
    from paper_1604_08501_amd import semvol
    if not os.path.exists(semvol.LIB_PATH):
        from paper_1604_08501_amd import build
        build.build()
    f = semvol.lib()._ZN6semapi20batch_default_shapesEibPKNS_10BatchOrderEiPNS_11DefaultTileE
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int32, ctypes.c_bool, ctypes.POINTER(Order), ctypes.c_int,
                  ctypes.POINTER(Tile)]

    def call(dtype, *blocks, rk=False):
        """(lanes, [(elements per tile, layout)]) of blocks (order, elements)."""
        orders = (Order * len(blocks))(*[Order(*b) for b in blocks])
        tiles = (Tile * len(blocks))()
        nt = f(dtype, rk, orders, len(blocks), tiles)
        return nt, [(t.epb, t.lay) for t in tiles]
    return call


@pytest.mark.parametrize("nq", [7, 8])
def test_few_nodes_keep_all_fluxes_resident(shapes, nq):
    last = 240000 // nq ** 3
    assert shapes(F64, (nq, last)) == (256, [(1, FULL)])
    assert shapes(F64, (nq, last + 1)) == (256, [(1, ALIAS)])
    assert shapes(F64, (nq, 1), rk=True) == (256, [(1, ALIAS)])
    assert shapes(F32, (nq, 1)) == (256, [(1, ALIAS)])


def test_other_orders_do_not_change_with_the_node_count(shapes):
    for nq in (5, 6, 9, 10):
        at = 240000 // nq ** 3
        assert shapes(F64, (nq, at)) == shapes(F64, (nq, at + 1)) == shapes(F64, (nq, 1))
    # the highest order of the batch decides
    for top in (6, 7, 8):
        assert shapes(F64, (4, 20), (top, 20)) == (256, [(8, FULL), (1, FULL)])
    for top in (5, 9):
        assert shapes(F64, (4, 20), (top, 20)) == shapes(F64, (4, 5000), (top, 5000))


def test_nq4_in_fp64_keeps_eight_elements_per_tile(shapes):
    assert shapes(F64, (4, 1)) == shapes(F64, (4, MAX_TILES * 8)) == (512, [(8, FULL)])
    assert shapes(F64, (4, 5000), (6, 5000)) == (512, [(8, FULL), (4, ALIAS)])
    assert shapes(F64, (4, 1), rk=True) == (256, [(4, FULL)])
    assert shapes(F32, (4, 1)) == (256, [(2, FULL)])


@pytest.mark.parametrize("dtype,nq,small,dense", [(F64, 2, 32, 64), (F32, 2, 32, 128),
                                                  (F32, 3, 8, 16)])
def test_dense_tiles_where_only_they_fit_the_table(shapes, dtype, nq, small, dense):
    assert shapes(dtype, (nq, MAX_TILES * small))[1] == [(small, FULL)]
    assert shapes(dtype, (nq, MAX_TILES * small + 1))[1] == [(dense, FULL)]
    assert shapes(dtype, (nq, MAX_TILES * dense))[1] == [(dense, FULL)]
    assert shapes(dtype, (nq, MAX_TILES * dense + 1))[1] == [(small, FULL)]   # a plan's only


def test_dense_tiles_of_several_orders(shapes):
    half = MAX_TILES // 2
    fits = ((2, half * 32), (3, half * 8))
    over = ((2, half * 32), (3, half * 8 + 1))
    assert shapes(F32, *fits)[1] == [(32, FULL), (8, FULL)]
    assert shapes(F32, *over)[1] == [(128, FULL), (16, FULL)]
    # two blocks of one order are counted apart: their tiles are not shared
    assert shapes(F32, (3, 8 * half - 1), (3, 8 * half - 1))[1] == [(8, FULL)] * 2
    assert shapes(F32, (3, 8 * half + 1), (3, 8 * half - 1))[1] == [(16, FULL)] * 2
