"""The library's rules by lattice size, called on the host without a GPU: which
passes a lattice takes, and with what launch."""
import ctypes

import pytest

prs = pytest.importorskip("paper_1710_10420_amd.prs")


class Geometry(ctypes.Structure):
    _fields_ = [("ndim", ctypes.c_int), ("f64", ctypes.c_int), ("nx", ctypes.c_int64), ("Q", ctypes.c_int64),
                ("M", ctypes.c_int64)]


class Tiling(ctypes.Structure):
    _fields_ = [("vec", ctypes.c_int), ("rows", ctypes.c_int), ("ty", ctypes.c_int)]


class BlkShape(ctypes.Structure):
    _fields_ = [("vec", ctypes.c_int), ("rows", ctypes.c_int), ("waves", ctypes.c_int), ("us", ctypes.c_float)]


class BlkGrid(ctypes.Structure):
    _fields_ = [("tiles_x", ctypes.c_int64), ("blocks", ctypes.c_int64), ("halo_lanes", ctypes.c_int32)]


class TileCounts(ctypes.Structure):
    _fields_ = [("x", ctypes.c_int64), ("q", ctypes.c_int64), ("s", ctypes.c_int64), ("ntiles", ctypes.c_int64)]


class PassChoice(ctypes.Structure):
    _fields_ = [("steps", ctypes.c_int), ("us", ctypes.c_float), ("blk", ctypes.c_bool), ("til", Tiling)]


def rule(name, res, *args):
    f = getattr(prs._lib, name)
    f.restype, f.argtypes = res, args
    return f


_G, _T, _I = ctypes.POINTER(Geometry), ctypes.POINTER(Tiling), ctypes.c_int
tb_supported = rule("_ZN3prs12tb_supportedERKNS_8GeometryE", ctypes.c_bool, _G)
blk_supported = rule("_ZN3prs13blk_supportedERKNS_8GeometryE", ctypes.c_bool, _G)
blk_choose = rule("_ZN3prs10blk_chooseERKNS_8GeometryEi", BlkShape, _G, _I)
blk_grid = rule("_ZN3prs8blk_gridERKNS_8GeometryEiiii", BlkGrid, _G, _I, _I, _I, _I)
auto_tile2 = rule("_ZN3prs10auto_tile2ERKNS_8GeometryEi", Tiling, _G, _I)
auto_step = rule("_ZN3prs9auto_stepERKNS_8GeometryE", PassChoice, _G)
tile_counts = rule("_ZN3prs11tile_countsERKNS_8GeometryERKNS_6TilingE", TileCounts, _G, _T)
auto_pass3 = rule("_ZN3prs10auto_pass3ERKNS_8GeometryEi", PassChoice, _G, _I)
auto_adj_tile = rule("_ZN3prs13auto_adj_tileERKNS_8GeometryEPi", Tiling, _G, ctypes.POINTER(ctypes.c_int))
tba_supported = rule("_ZN3prs13tba_supportedERKNS_8GeometryERKNS_6TilingEi", ctypes.c_bool, _G, _T, _I)
tb_tiles = rule("_ZN3prs8tb_tilesERKNS_8GeometryERKNS_6TilingEi", ctypes.c_int64, _G, _T, _I)


def geometry(shape, f64=False):
    return Geometry(len(shape), int(f64), shape[0], shape[1] if len(shape) == 3 else 1, shape[-1])


WORK_ITEMS = 2 ** 32      # a launch holds fewer


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(2 ** 28 - 1, 1), (1, 10 ** 9), (3, 8 * 10 ** 8), (1, 2 ** 30), (64, 2 ** 24),
                                   (8192, 8192)])
def test_block_passes_fit_a_launch(shape, f64):
    g = geometry(shape, f64)
    assert tb_supported(g)
    for steps in range(1, 17):
        b = blk_choose(g, steps)
        if b.vec == 0:
            continue
        n = blk_grid(g, b.vec, b.rows, b.waves, steps).blocks
        assert 0 < n * b.waves * 64 < WORK_ITEMS, (steps, b.vec, b.rows, b.waves, n)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(2047, 2047), (2048, 2048), (1023, 4095), (8191, 8191), (1, 10 ** 6), (255, 255),
                                   (301, 640)])
def test_default_2d_tiles_grow_with_the_lattice(shape, f64):
    """Three tiles per SIMD are enough (1024 SIMDs); beyond, a tile grows to 32
    rows (64 with two sites a lane): at 8 rows an eight-step pass marches 22
    rows for the 8 it stores."""
    g = geometry(shape, f64)
    for T in (2, 8):
        t = auto_tile2(g, T)
        assert shape[0] % t.vec == 0
        assert t.rows == (32 if t.vec == 1 else 64) or tb_tiles(g, t, T) <= 3072, (T, t.vec, t.rows)


@pytest.mark.parametrize("shape,us", [((512, 512), 5.4), ((2048, 2048), 14.0), ((1, 100000), 21.5), ((30, 100000), 25.3),
                                      ((61, 60000), 20.6)])
def test_single_step_estimate_counts_narrow_rows(shape, us):
    """Timed single steps (default tiles, float32), within a third; and two of
    them do not stand before a block pass of two steps on a narrow lattice,
    where a block pass takes about 15 us."""
    g = geometry(shape)
    assert us / 1.33 < auto_step(g).us < us * 1.33
    assert blk_choose(g, 2).us < 2 * auto_step(g).us


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 6 * 10 ** 8), (1, 1, 2 ** 31 - 2 ** 14), (2, 2, 10 ** 9), (5, 3, 6 * 10 ** 8),
                                   (1, 1, 1), (64, 64, 64), (1024, 1024, 1024)])
def test_3d_passes_fit_a_launch(shape, f64):
    g = geometry(shape, f64)
    for T in (2, 3, 4, 5):
        c = auto_pass3(g, T)
        if c.til.vec:
            assert tb_tiles(g, c.til, T) * 64 < WORK_ITEMS, (T, c.til.rows)
    T = ctypes.c_int()
    t = auto_adj_tile(g, T)
    if tba_supported(g, t, T.value):
        assert tb_tiles(g, t, T.value) * 64 < WORK_ITEMS


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(2 ** 28 - 1, 1), (1, 10 ** 9), (1, 2 ** 30), (2, 10 ** 9), (1, 1, 6 * 10 ** 8),
                                   (1, 1, 2 ** 31), (1, 1, 2 ** 33), (1, 2 ** 33)])
def test_default_single_steps_fit_a_launch(shape, f64):
    g = geometry(shape, f64)
    assert tile_counts(g, auto_step(g).til).ntiles * 64 < WORK_ITEMS
    if len(shape) == 2 and tb_supported(g):
        for T in (2, 8):
            t = auto_tile2(g, T)
            assert tile_counts(g, t).ntiles * 64 < WORK_ITEMS and tb_tiles(g, t, T) * 64 < WORK_ITEMS


@pytest.mark.parametrize("shape", [(1, 1, 2 ** 31), (1, 1, 2 ** 31 - 2 ** 13), (1, 1, 2 ** 33), (1, 2 ** 31), (1, 2 ** 33)])
def test_rows_past_32_bits_run_single_steps(shape):
    """The multi-step passes count rows (2D) and planes (3D) in 32 bits."""
    assert not tb_supported(geometry(shape))


auto_adj_step = rule("_ZN3prs13auto_adj_stepERKNS_8GeometryE", Tiling, _G)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(16, 16), (2048, 2048), (4096, 4096), (4095, 4095), (1, 10 ** 9), (33, 50, 21),
                                   (256, 256, 256), (255, 255, 255), (1, 1, 2 ** 33)])
def test_single_reverse_steps_have_a_tiling_of_their_own(shape, f64):
    """Short tiles with 16 bytes a lane on large lattices, whatever the reverse
    passes take, in a launch that holds them."""
    g = geometry(shape, f64)
    t = auto_adj_step(g)
    assert shape[0] % t.vec == 0 and tile_counts(g, t).ntiles * 64 < WORK_ITEMS
    field = g.nx * g.Q * g.M * (8 if f64 else 4)
    widest = 4 if shape[0] % 4 == 0 and not f64 else 2 if shape[0] % 2 == 0 else 1
    assert t.vec == (widest if field >= 4e6 else 1)
    assert t.rows in (8, 16) or tile_counts(g, Tiling(t.vec, 16, t.ty)).ntiles * 64 >= WORK_ITEMS


@pytest.mark.parametrize("shape,T", [((1, 1, 20000), 1), ((64, 1, 2000), 4), ((64, 64, 64), 4), ((10, 10, 1000), 4)])
def test_lattices_of_a_few_rows_take_single_reverse_steps(shape, T):
    """1 x 1 x 20000: 33 us a step in passes of two, 9 in single steps."""
    n = ctypes.c_int()
    auto_adj_tile(geometry(shape), n)
    assert n.value == T
