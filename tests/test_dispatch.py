"""Host logic: which kernels slope_spmm_fwd picks for a shape (slope_spmm_fwd_plan, no GPU needed).
The regimes pinned here are the ones the design notes describe; the boundaries are properties of the
cost estimates, not of measured times."""
import time

import pytest

from paper_2405_16325_amd import binding as sl

STREAM, SLABS, TILE, GENERIC, STREAM_ROWS, TILE_AND_STREAM = range(6)


@pytest.mark.parametrize("b", [1, 7, 16, 17, 32])
@pytest.mark.parametrize("d_out,d_in", [(9216, 9216), (36864, 9216), (9216, 36864), (512, 128)])
def test_up_to_32_tokens_take_a_small_batch_kernel(b, d_out, d_in):
    p = sl.slope_spmm_fwd_plan(b, d_in, d_out)
    assert p["product"] in (STREAM, STREAM_ROWS)
    assert p["tokens"] == (16 if b <= 16 else 32)
    if p["product"] == STREAM:
        assert p["slabs"] == 1 and p["rows"] in ((32, 48, 64) if b <= 16 else (32, 48))
    else:
        assert p["rows"] == 48 and d_in % 1024 == 0 and p["slabs"] * -(-d_out // 48) >= 512


def test_row_split_form_of_the_small_batch_kernel():
    # a tall matrix: one workgroup per 48 rows fills the chip three times, no slices
    p = sl.slope_spmm_fwd_plan(16, 9216, 36864)
    assert (p["product"], p["slabs"]) == (STREAM_ROWS, 1)
    assert sl.slope_spmm_fwd_plan(16, 9216, 36864, 0, False)["product"] == STREAM_ROWS
    # 192 workgroups and a long contraction (36 chunks of 1024): cut into 4 slices with scratch, else the kernel
    # whose wavefronts split the contraction; 9 chunks are too few to pay for the second launch
    p = sl.slope_spmm_fwd_plan(16, 36864, 9216)
    assert (p["product"], p["slabs"]) == (STREAM_ROWS, 4)
    assert sl.slope_spmm_fwd_plan(16, 36864, 9216, 0, False)["product"] == STREAM
    assert sl.slope_spmm_fwd_plan(16, 9216, 9216)["product"] == STREAM
    # 17 to 32 tokens: only where a long contraction over few rows wants four slices or more
    assert sl.slope_spmm_fwd_plan(32, 36864, 9216)["product"] == STREAM_ROWS
    assert sl.slope_spmm_fwd_plan(32, 9216, 9216)["product"] == STREAM
    assert sl.slope_spmm_fwd_plan(32, 9216, 36864)["product"] == STREAM
    # 625 workgroups fill the chip without slices, which 9 chunks would not pay for: the same with and without scratch
    assert [sl.slope_spmm_fwd_plan(16, 9216, 30000, 0, ws)["slabs"] for ws in (True, False)] == [1, 1]
    assert sl.slope_spmm_fwd_plan(16, 9216, 30000)["product"] == STREAM_ROWS
    # contractions that are no multiple of 1024, and matrices too small to fill the chip either way
    assert sl.slope_spmm_fwd_plan(16, 2560, 36864)["product"] == STREAM
    assert sl.slope_spmm_fwd_plan(16, 1024, 2048)["product"] == STREAM


def test_small_batch_rows_avoid_a_thin_last_round():
    # 9216 rows: 288 workgroups of 32 rows would leave a last round of 32; 192 of 48 rows fit one round
    assert sl.slope_spmm_fwd_plan(1, 9216, 9216, 0, False)["rows"] == 48
    # 8192 rows: 256 workgroups of 32 rows are exactly one round
    assert sl.slope_spmm_fwd_plan(1, 9216, 8192, 0, False)["rows"] == 32


def test_contraction_shorter_than_two_k_steps_stays_off_the_small_batch_kernel():
    assert sl.slope_spmm_fwd_plan(4, 64, 512)["product"] != STREAM


@pytest.mark.parametrize("b", [33, 100, 128, 200, 256])
def test_mid_batches_split_the_contraction_only_with_scratch_and_few_tiles(b):
    with_ws = sl.slope_spmm_fwd_plan(b, 9216, 9216, 0, True)
    without = sl.slope_spmm_fwd_plan(b, 9216, 9216, 0, False)
    assert with_ws["product"] == SLABS and with_ws["slabs"] >= 2 and with_ws["rows"] == 256
    assert without["product"] == TILE and without["slabs"] == 1
    # 36864 weight rows and two token tiles: 288 tiles fill the chip, no split
    big = sl.slope_spmm_fwd_plan(b, 9216, 36864, 0, True)
    assert (big["product"] == SLABS) == (b <= 128)


@pytest.mark.parametrize("b,d_out,d_in,slabs", [(64, 9984, 7168, True), (64, 12288, 12288, True), (128, 7168, 7168, True), (64, 12544, 20480, True),
                                                (64, 4096, 2048, False), (128, 4096, 4096, False), (48, 16384, 5120, False)])
def test_long_contractions_split_although_64_x_64_tiles_fit_a_round(b, d_out, d_in, slabs):
    assert -(-d_out // 64) * -(-b // 64) <= 256
    assert (sl.slope_spmm_fwd_plan(b, d_in, d_out)["product"] == SLABS) == slabs


def test_slabs_times_tiles_fits_one_round_for_two_token_tiles():
    p = sl.slope_spmm_fwd_plan(256, 9216, 9216, 0, True)       # 36 x 2 tiles
    assert p["slabs"] == 3                                      # 216 workgroups: one round; 4 slabs would need two


@pytest.mark.parametrize("b,d_out,d_in", [(16384, 9216, 9216), (16384, 36864, 9216), (16384, 9216, 36864)])
def test_large_training_shapes_take_the_largest_tile(b, d_out, d_in):
    p = sl.slope_spmm_fwd_plan(b, d_in, d_out, 0, True)
    assert p["product"] == TILE and (p["rows"], p["tokens"]) == (256, 256) and p["slabs"] == 1


def test_a_small_layer_gets_a_tile_that_fits_one_round():
    p = sl.slope_spmm_fwd_plan(2048, 768, 3072, 0, True)       # OPT-125m fc1
    tiles = -(-3072 // p["rows"]) * -(-2048 // p["tokens"])
    assert p["product"] == TILE and tiles <= 256


def test_contractions_by_their_multiple_of_64():
    # on one round of 64 x 64 tiles only whole pairs of k-steps count as a tile shape
    assert sl.slope_spmm_fwd_plan(300, 320, 448)["product"] == GENERIC
    assert sl.slope_spmm_fwd_plan(300, 512, 448)["product"] == TILE
    # on more tiles whole k-steps do, at least two of them
    assert sl.slope_spmm_fwd_plan(3000, 320, 4480)["product"] == TILE
    assert sl.slope_spmm_fwd_plan(3000, 328, 4480)["product"] == GENERIC
    assert sl.slope_spmm_fwd_plan(3000, 64, 4480)["product"] == GENERIC


# where the estimate takes a round of 64 x 64 tiles for more than 16 k-steps: 128 x 64 for an odd number of them, from 2.5 MB of operands on, with an
# adapter from 5 MB on
@pytest.mark.parametrize("b,d_out,d_in,plain,adapter", [
    (200, 768, 1152, 64, 64), (112, 512, 1280, 64, 64), (300, 1024, 1792, 128, 64), (600, 512, 2304, 128, 64), (1300, 512, 1792, 128, 128),
    (67, 5888, 2560, 128, 128), (43, 4160, 1728, 128, 128), (86, 256, 1344, 128, 128), (300, 64, 1344, 0, 0), (300, 1024, 1024, 64, 64)])
def test_rows_of_a_tile_where_a_round_of_64_x_64_is_estimated(b, d_out, d_in, plain, adapter):
    for r, rows in ((0, plain), (32, adapter), (160, adapter)):
        p = sl.slope_spmm_fwd_plan(b, d_in, d_out, r, False)
        assert (p["product"], p["rows"], p["tokens"]) == ((TILE, rows, 64) if rows else (GENERIC, 64, 64))


@pytest.mark.parametrize("b,d_out,d_in", [(33, 16640, 1024), (64, 20480, 1024), (64, 20480, 1088), (64, 25344, 576)])
def test_more_than_a_round_of_64_x_64_tiles_stays_on_the_tile_kernel(b, d_out, d_in):
    assert -(-d_out // 64) > 256
    p = sl.slope_spmm_fwd_plan(b, d_in, d_out, 0, False)
    assert (p["product"], p["rows"], p["tokens"]) == (TILE, 128, 64)
    assert sl.slope_spmm_fwd_plan(b, d_in, 36864, 0, False)["rows"] == 192


def test_a_few_tokens_beyond_whole_tiles_take_the_small_batch_kernel():
    def plan(b, d_out, d_in, r=0):
        p = sl.slope_spmm_fwd_plan(b, d_in, d_out, r)
        return p["product"], p["rows"], p["tokens"], p["slabs"]
    # 80 x 3 tiles of 256 x 256 are a round, the nine tokens left would begin another
    assert plan(777, 20480, 5120, 64) == (TILE_AND_STREAM, 256, 256, 9)
    assert plan(768, 20480, 5120)[0] == TILE
    assert plan(800, 20480, 5120) == (TILE_AND_STREAM, 256, 256, 32) and plan(801, 20480, 5120)[0] == TILE
    assert plan(4097, 4096, 2112) == (TILE_AND_STREAM, 256, 256, 1)
    assert plan(16385, 36864, 9216)[0] == TILE                          # a pass over this weight costs more than the round


def test_short_adapter_products_of_many_tokens():
    xl = lambda b, d_in, r: sl.slope_spmm_fwd_plan(b, d_in, 2048, r)["xl"]
    assert xl(1024, 1280, 64) == 4 and xl(1024, 1344, 64) != 4           # five chunks of 32 rows of L per wavefront and six, 32 tiles
    assert xl(2048, 1536, 64) == 4 and xl(2048, 1600, 64) != 4           # six and seven, 64 tiles
    assert xl(8192, 1024, 64) == 4 and xl(8224, 1024, 64) != 4           # one round of tiles and a tile more
    assert xl(512, 2048, 64) == 1


def test_split_of_a_partial_round_by_slabs():
    slabs = lambda b, d_out, d_in: sl.slope_spmm_fwd_plan(b, d_in, d_out)["slabs"]
    assert slabs(530, 1792, 4864) >= 2 and slabs(512, 2048, 8192) >= 2
    # measured as fast or faster whole: one launch, no scratch (26.6 us against 27.3; 21 us against 24)
    assert slabs(700, 2112, 4160) == 1 and slabs(512, 4096, 4096) == 1 and slabs(1024, 2048, 4096) == 1
    assert slabs(700, 2112, 960) == 1                                    # fewer than four quads of k-steps per slab
    assert slabs(2048, 768, 3072) == 1                                   # a microsecond slower in a step
    assert sl.slope_spmm_fwd_plan(700, 4160, 2112, 0, False)["slabs"] == 1


# whatever the tile: a caller that looks for code 1 finds every product that wants the workspace for slabs
@pytest.mark.parametrize("b,d_out,d_in,r,rows", [(33, 520, 8192, 32, 128), (34, 3328, 4160, 0, 128), (38, 3072, 6400, 256, 128), (67, 4176, 4096, 0, 192),
                                                 (64, 9216, 9216, 128, 256), (300, 2304, 5120, 160, 192)])
def test_every_split_product_has_one_code(b, d_out, d_in, r, rows):
    p = sl.slope_spmm_fwd_plan(b, d_in, d_out, r)
    assert (p["product"], p["rows"]) == (SLABS, rows) and p["slabs"] > 1


def test_long_weights_on_too_few_rows_of_256_are_filled_up_with_smaller_tiles():
    # 16 x 4 and 32 x 2 tiles of 256 x 128 in the three slabs there is room for are 192 workgroups
    for b, d_out, d_in in ((482, 4096, 8192), (134, 8064, 7808), (217, 512, 19456)):
        p = sl.slope_spmm_fwd_plan(b, d_in, d_out)
        assert p["product"] == SLABS and p["rows"] < 256
    assert sl.slope_spmm_fwd_plan(128, 9216, 9216)["rows"] == 256


def test_adapter_beside_a_split_product_does_not_outlast_it():
    def plan(b, d_out, d_in, r):
        p = sl.slope_spmm_fwd_plan(b, d_in, d_out, r)
        return p["rows"], p["tokens"], p["slabs"]
    # in eight slabs of 128 x 64 the 16 compute units left over would take 53 chunks of X L for 56 k-steps of the product
    assert plan(166, 1280, 27008, 0) != plan(166, 1280, 27008, 32)
    # 234 workgroups are 30 on most XCDs: the last of 22 for X L would be a 33rd there and wait for the round to end
    assert plan(330, 3328, 13568, 64) == (256, 128, 5)


def test_adapter_product_regimes():
    xl = lambda b, r=128, d_in=9216: sl.slope_spmm_fwd_plan(b, d_in, 9216, r)["xl"]
    assert sl.slope_spmm_fwd_plan(64, 9216, 9216, 0)["xl"] == 0
    assert [xl(b) for b in (1, 16, 17, 128, 512)] == [1] * 5    # split over d_in, L as stored
    assert [xl(b) for b in (513, 4096)] == [3, 3]               # dense tile kernel, too few tiles: split over d_in
    assert xl(16384) == 2                                       # 256 tiles: no split
    # chunks of 64 rows of L per partial sum that the scratch is sized by: as many as still give 256 workgroups
    chunks = lambda b, d_in: sl.slope_spmm_fwd_plan(b, d_in, 9216, 128)["xl_chunks"]
    assert chunks(16, 9216) == 1 and chunks(64, 9216) == 1 and chunks(16, 36864) == 2 and chunks(512, 36864) == 4


@pytest.mark.parametrize("b,d_out,d_in,r", [(128, 4096, 4096, 128), (300, 4096, 4096, 0), (700, 2112, 4160, 0)])
def test_planning_costs_less_than_the_call_into_the_library(b, d_out, d_in, r):
    """Every call plans, and the small ones are bound by the host: the query of a shape against one that plans nothing
    (0.55 us through ctypes, 0.1 to 0.3 more here; 1.5 to 1.9 more while every form was priced)."""
    query = sl.lib().slope_spmm_fwd_workspace_bytes

    shapes, best = ((b, d_in, d_out, r), (0, d_in, d_out, r)), [float("inf")] * 2
    for _ in range(200):
        for i, shape in enumerate(shapes):                                   # in turn: the machine's speed may drift
            t = time.perf_counter()
            for _ in range(100):
                query(*shape)
            best[i] = min(best[i], time.perf_counter() - t)
    assert best[0] < 2.5 * best[1]


def test_plan_rejects_what_the_call_rejects():
    with pytest.raises(sl.SlopeError):
        sl.slope_spmm_fwd_plan(0, 9216, 9216)
    with pytest.raises(sl.SlopeError):
        sl.slope_spmm_fwd_plan(16, 9216, 9216, 48)
    with pytest.raises(sl.SlopeError):
        sl.slope_spmm_fwd_plan(16, 9204, 9216)


def test_extents_that_are_not_multiples_of_64_take_the_general_kernels():
    # any multiple of 8 is accepted; a contraction that is not a whole number of k-steps of 64 goes to the
    # generic kernel's form for ragged rows (also for inference-size batches) and to the kernel for ragged extents for X L
    for b in (1, 16, 300, 5000):
        plan = sl.slope_spmm_fwd_plan(b, 1000, 1000, 64)
        assert plan["product"] == GENERIC and plan["xl"] == 4
    assert sl.slope_spmm_fwd_plan(16, 1024, 1000, 64)["product"] == 0      # d_out may be ragged on the fast paths
    assert sl.slope_spmm_fwd_plan(4096, 1024, 1000, 64)["product"] == TILE
