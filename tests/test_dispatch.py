"""The choice between the two forms of the large-batch kernel: host code, no GPU needed.  Pairs (1, 100) and above are the level form
(weights by look-up), every other pair is the summing form."""
import ctypes

import pytest

import paper_2510_10467_amd as bcq
from paper_2510_10467_amd import build as hip_build


@pytest.fixture(scope="module", autouse=True)
def built():
    if hip_build.is_stale():
        hip_build.build()


@pytest.fixture
def knobs():
    yield
    bcq.select_dequant_shape(0, 0)
    bcq.select_kernel("auto")


def takes_level_form(p, m, n, batch, group=128, with_offsets=False):
    tiles, blocks = bcq.dequant_shape_for(p, m, n, batch, group, with_offsets)
    return tiles == 1 and blocks >= 100


# (p, m, n, batch, group, offsets): microseconds on one MI355X of the summing form and of the level form's best shape for that call
SUMMING_IS_AHEAD = [
    ((4, 13824, 256, 90, 256, True), 5.8, 6.3),         # what a round takes at any width decides on narrow matrices
    ((2, 6144, 256, 105, 128, False), 4.3, 5.1),
    ((4, 4864, 256, 153, 64, False), 5.1, 5.8),
    ((2, 2816, 512, 229, 64, True), 5.5, 6.2),
    ((4, 11542, 1024, 46, 64, True), 9.4, 10.9),
    ((4, 1024, 1280, 320, 128, False), 7.3, 9.1),       # widths that leave the teams of a workgroup unequal shares
    ((4, 4096, 1280, 128, 128, False), 8.0, 9.7),
    ((4, 16655, 1024, 276, 128, True), 31.3, 35.0),     # sixteen levels
    ((4, 5289, 11520, 955, 128, True), 246.9, 254.4),
    ((4, 13824, 18688, 497, 256, True), 424.8, 478.0),
]

LEVEL_IS_AHEAD = [
    ((3, 28672, 8192, 2048, 128, False), 1182.0, 917.0),
    ((4, 8192, 8192, 96, 64, False), 48.0, 38.3),
    ((3, 8935, 8960, 211, 128, False), 103.0, 75.4),
    ((4, 5632, 26624, 189, 64, False), 195.7, 157.6),
    ((4, 3208, 16384, 365, 128, False), 127.5, 100.9),
    ((2, 9397, 3584, 184, 128, True), 32.2, 22.4),
    ((1, 17408, 27904, 161, 128, True), 343.9, 231.0),
]


@pytest.mark.parametrize("call,summing_us,level_us", SUMMING_IS_AHEAD)
def test_summing_form_where_it_is_ahead(call, summing_us, level_us):
    assert not takes_level_form(*call)


@pytest.mark.parametrize("call,summing_us,level_us", LEVEL_IS_AHEAD)
def test_level_form_where_it_is_ahead(call, summing_us, level_us):
    assert takes_level_form(*call)


# ((precisions), m, n, batch, group, offsets): microseconds of the form that rebuilds weights by sums and of the level form
@pytest.mark.parametrize("call,summing_us,level_us", [
    (((2, 3, 4), 11520, 256, 45, 64, False), 10.1, 12.7),               # up to 64 requests: a second round of workgroups
    (((2, 3, 4), 13312, 512, 64, 64, False), 13.8, 15.4),
    (((2, 3, 4), 16128, 768, 41, 64, True), 17.7, 19.8),
    (((1, 2, 3, 4), 12288, 256, 47, 64, False), 10.6, 12.3),
    (((2, 3, 4), 17433, 768, 196, 64, False), 25.5, 33.4),              # beyond: two workgroups of 128 x 128 on a CU
    (((2, 3, 4), 21760, 768, 228, 64, False), 30.2, 42.1)])
def test_summing_forms_where_they_are_ahead_with_per_request_precision(call, summing_us, level_us):
    assert bcq.mixed_shape_for(*call) == (0, 0)


@pytest.mark.parametrize("call,summing_us,level_us", [
    (((2, 3, 4), 9472, 256, 49, 64, False), 10.3, 8.2),
    (((2, 3, 4), 19363, 256, 62, 64, False), 17.7, 13.7),
    (((2, 3, 4), 18176, 768, 47, 64, False), 26.8, 19.4),
    (((2, 3, 4), 21498, 1024, 42, 64, False), 33.1, 22.9),
    (((2, 3, 4), 4956, 2816, 52, 64, False), 46.4, 18.4),
    (((2, 3, 4), 8192, 8192, 200, 128, False), 118.6, 63.0)])
def test_level_form_where_it_is_ahead_with_per_request_precision(call, summing_us, level_us):
    assert bcq.mixed_shape_for(*call)[0] == 1


def test_per_request_precision_that_the_level_form_does_not_take(knobs):
    assert bcq.mixed_shape_for((2, 3, 4), 8192, 8192, 32) == (0, 0)             # one tile of 32 requests
    assert bcq.mixed_shape_for((2, 3, 4), 8192, 8192 + 128, 200) == (0, 0)      # not whole pairs of column groups
    for bad in (((), 8192, 8192, 200), ((5,), 8192, 8192, 200), ((2,), 8192, 8192, 200, 32), ((2,), 0, 8192, 200), ((2,), 8192, 8192, 0)):
        with pytest.raises(bcq.BcqError) as error:
            bcq.mixed_shape_for(*bad)
        assert error.value.status == -6
    assert bcq.lib().bcq_mixed_shape_for(4, 8192, 8192, 200, 128, 0, None, None) == -1
    automatic = bcq.mixed_shape_for((2, 3, 4), 1024, 1024, 100), bcq.mixed_shape_for((2, 3, 4), 8192, 8192, 200)
    assert automatic == ((0, 0), (1, 96))
    for blocks in (96, 101, 105):
        bcq.select_dequant_shape(1, blocks)
        assert bcq.mixed_shape_for((2, 3, 4), 1024, 1024, 100) == (1, blocks)
        assert bcq.mixed_shape_for((2, 3, 4), 1024, 1152, 100) == (0, 0)
    bcq.select_dequant_shape(1, 100)                                            # not a shape of these calls
    assert (bcq.mixed_shape_for((2, 3, 4), 1024, 1024, 100), bcq.mixed_shape_for((2, 3, 4), 8192, 8192, 200)) == automatic
    bcq.select_dequant_shape(1, 96)                                             # and one of these calls only
    with pytest.raises(bcq.BcqError) as error:
        bcq.dequant_shape_for(4, 8192, 8192, 200)
    assert error.value.status == -6
    bcq.select_dequant_shape(4, 8)
    assert bcq.mixed_shape_for((2, 3, 4), 8192, 8192, 200) == (0, 0)


def test_what_the_level_form_does_not_take():
    assert takes_level_form(4, 28672, 8192, 33)
    assert not takes_level_form(4, 28672, 8192, 32)             # one tile of 32 requests
    assert takes_level_form(4, 28672, 8192, 500)
    assert not takes_level_form(4, 28672, 8192 + 128, 500)      # not whole pairs of column groups
    for bad in ((5, 28672, 8192, 500, 128), (4, 28672, 8192, 500, 32), (0, 28672, 8192, 500, 128), (4, 0, 8192, 500, 128), (4, 28672, 8192, 0, 128)):
        with pytest.raises(bcq.BcqError) as error:              # five planes, groups of 32, no problem at all
            bcq.dequant_shape_for(*bad)
        assert error.value.status == -6
    assert bcq.lib().bcq_dequant_shape_for(4, 28672, 8192, 500, 128, 0, None, None) == -1


def test_forced_level_form_refuses_what_it_does_not_take(knobs):
    """A forced shape that cannot run the problem is reported as that (-6) before anything is launched (made-up addresses do), from
    every entry point.  (Per-request precision runs on its other kernels there, see the test of its forced shapes.)"""
    L = bcq.lib()
    P, S, X, Y = 0x10000, 0x20000, 0x30000, 0x40000
    bcq.select_kernel("dequant_mfma")
    bcq.select_dequant_shape(1, 102)
    assert L.bcq_gemv(P, S, 3, X, Y, 4096, 640, 70, 128, None) == -6
    assert L.bcq_gemv_offset(P, S, S, 3, X, Y, 4096, 640, 70, 128, None) == -6
    assert L.bcq_dequant_shape_for(3, 4096, 640, 70, 128, 0, ctypes.byref(ctypes.c_int()), ctypes.byref(ctypes.c_int())) == -6
    pp = (ctypes.c_void_p * 2)(P, P + 0x1000)
    sp = (ctypes.c_void_p * 2)(S, S + 0x1000)
    yp = (ctypes.c_void_p * 2)(Y, Y + 0x1000)
    assert L.bcq_gemv_multi(2, pp, sp, (ctypes.c_int64 * 2)(4096, 4096), yp, 3, X, 640, 70, 128, None) == -6
    bcq.select_kernel("auto")
    assert L.bcq_gemv(P, S, 3, X, Y, 14336, 640, 70, 128, None) == -6


def test_a_refused_shape_changes_nothing(knobs):
    for forced in ((1, 103), (4, 8), (32, 2)):
        bcq.select_dequant_shape(*forced)
        for refused in ((3, 4), (1, 106), (1, 99), (-1, 4), (7, 7), (2, 100)):
            with pytest.raises(bcq.BcqError):
                bcq.select_dequant_shape(*refused)
            assert bcq.dequant_shape_for(4, 28672, 8192, 500) == forced
    bcq.select_dequant_shape(0, 0)
    assert bcq.dequant_shape_for(4, 28672, 8192, 500) not in ((1, 103), (4, 8), (32, 2))


# (row blocks of the shape, group, n): loads a plane of scales takes before the first weight, each of 256 bytes
@pytest.mark.parametrize("blocks,group,n,loads", [
    (104, 128, 256, 2), (104, 64, 256, 4), (104, 256, 256, 2), (104, 128, 512, 4), (104, 256, 768, 4), (104, 128, 1024, 8),
    (103, 128, 256, 1), (103, 256, 256, 1), (103, 64, 512, 4), (101, 128, 256, 2), (100, 256, 512, 4)])
def test_a_window_of_scales_is_no_wider_than_the_matrix(blocks, group, n, loads):
    """A row of 256 columns in groups of 128 has four bytes of scales per plane: 64 rows in one load, not four (64 x 128, p = 4 with
    offsets: 9.4 us with 80 loads ahead of the first weight, 8.4 with five)."""
    for p in (1, 2, 3, 4):
        assert bcq.level_layout(p, blocks, n, group, False)["window_loads"] == p * loads
        if blocks != 104:                                       # (where every lane reads its own offset at p = 4)
            assert bcq.level_layout(p, blocks, n, group, True)["window_loads"] == (p + 1) * loads


def test_windows_in_groups_of_256_are_whole_where_nothing_is_cut_off():
    """A scale is two bytes; rows of an odd number of them start at odd multiples of two bytes every other time, between dwords."""
    for p in (1, 2, 3, 4):
        for offsets in (False, True):
            window = 2 * bcq.level_layout(p, 103, 28672, 64, offsets)["window_columns"] // 64       # bytes of a row: two per group
            whole = 256 * (window // 2)
            columns = lambda n: bcq.level_layout(p, 103, n, 256, offsets)["window_columns"]
            assert columns(28672) == whole                      # 112 groups: every row starts at a multiple of four bytes
            assert columns(28672 - 256) == whole // 2           # 111
            assert columns(whole - 256) == whole                # one group less than a window has place for: the row fits with what lies before it
            assert columns(whole + 256) == whole // 2


def test_words_for_two_pairs_of_groups_at_a_time_only_where_that_is_ahead():
    columns = lambda p, blocks, n, offsets=False: bcq.level_layout(p, blocks, n, 128, offsets)["word_columns"]
    for n in (1536, 5120, 14336):
        for blocks in (101, 102):
            assert [columns(p, blocks, n) for p in (1, 2, 3, 4)] == [256, 256, 512, 512] and columns(4, blocks, n, True) == 256
        for blocks in (100, 104):
            assert {columns(p, blocks, n) for p in (1, 2, 3, 4)} == {256}
        for blocks in (103, 105):
            assert {columns(p, blocks, n) for p in (1, 2, 3, 4)} == {512 if n > 5120 else 256} and columns(4, blocks, n, True) == 256


def test_layout_refuses_what_the_form_does_not_take():
    for bad in ((5, 104, 512), (0, 104, 512), (4, 99, 512), (4, 106, 512), (4, 104, 384), (4, 104, 512, 32), (4, 104, 512, 512)):
        with pytest.raises(bcq.BcqError) as error:
            bcq.level_layout(*bad)
        assert error.value.status == -6
    assert bcq.lib().bcq_level_layout(4, 104, 512, 128, 0, None) == -1
