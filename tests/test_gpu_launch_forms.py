"""The forms that the launchers choose by the size of the launch, at the edges where each begins or ends, against the
float64 oracle and with guard zones around every output."""
import numpy as np
import pytest

from paper_1805_08899_amd.workloads import Workload, make_inputs
from parity import assert_parity, oracle_outputs, put_rows

pytestmark = pytest.mark.gpu

CASES = [
    # name, B, Tq, Tk, H, Dv, dtype, big (entries beyond the range of the factorised exponential)
    # recomputation, every tanh twice (few blocks): slices of 16, 32 and 64 columns, remainders on both axes, one row,
    # more rows than one staged range of dS, entries that need the exponential of the sum
    ("split_16_columns", 1, 33, 53, 12, 8, "f32", True),
    ("split_32_columns_ragged_h", 3, 130, 70, 90, 8, "f32", False),
    ("split_64_columns", 2, 61, 83, 256, 12, "f32", True),
    ("split_one_query", 2, 1, 70, 64, 8, "f32", False),
    ("split_one_key", 3, 70, 1, 40, 4, "f32", False),
    ("split_many_ranges", 1, 700, 300, 20, 4, "f32", False),
    ("split_bf16", 2, 37, 261, 100, 8, "bf16", False),
    # few blocks of the other form, but more groups of query rows than a grid holds: that form, in passes
    ("split_groups_past_a_grid", 1, 530000, 32, 4, 4, "f32", False),
    # recomputation with slices of 16 columns (four lane groups): rows not a multiple of four, more than one pass of 256
    # rows; 32 columns: fewer rows than lane groups would like, two passes; the whole of a narrow H in one slice
    ("slices_of_16", 25, 50, 21, 130, 8, "f32", True),
    ("slices_of_16_two_passes", 14, 259, 19, 240, 8, "f32", False),
    ("slices_of_16_bf16", 30, 35, 30, 112, 8, "bf16", False),
    # more than one round of blocks: 16 columns with one and two passes and a masked tail of H, 32 columns
    ("slices_of_16_two_rounds", 60, 140, 67, 201, 4, "f32", True),
    ("slices_of_16_two_rounds_two_passes", 67, 259, 21, 130, 4, "bf16", False),
    ("slices_of_32_two_rounds", 64, 100, 66, 300, 4, "f32", False),
    ("slices_of_32", 34, 45, 9, 470, 8, "f32", True),
    ("slices_of_32_two_passes", 20, 131, 9, 800, 4, "f32", False),
    ("slice_of_16_is_the_whole_h", 200, 9, 11, 16, 4, "f32", False),
    ("slice_of_32_is_the_whole_h", 200, 9, 11, 31, 4, "f32", False),
    # recomputation with up to 25 rows per lane: its fewest rows and the next ones that do not take it, odd
    # rows, columns and keys, all counts of keys in the first step, two lane groups and one, one to three passes, numbers of rows that
    # do and do not deal evenly; entries beyond the factor limit in the first step and in a later one
    ("rows_of_25_two_groups_60", 125, 60, 47, 130, 4, "f32", True),
    ("rows_of_25_not_59", 125, 59, 47, 130, 4, "f32", False),
    ("rows_of_25_72_bf16", 182, 72, 29, 128, 4, "bf16", False),
    ("rows_of_25_two_groups_100", 199, 100, 29, 127, 4, "f32", True),
    ("rows_of_25_one_group_101_bf16", 150, 101, 20, 185, 8, "bf16", False),
    ("rows_of_25_one_group_130", 202, 130, 13, 126, 4, "f32", True),
    ("rows_of_25_one_group_200", 221, 200, 13, 128, 4, "f32", False),
    ("rows_of_25_two_passes", 236, 201, 13, 99, 4, "f32", True),
    ("rows_of_25_three_passes", 447, 405, 8, 48, 4, "f32", False),
    # forward: blocks of four rows (eight waves, four waves), of eight rows with slices of 64 and 128 columns; a small batch
    # spread over the XCDs; H that is no multiple of four (tails of one to three columns, in both storage types), H of a
    # single group of four and just past it
    ("forward_four_rows_eight_waves", 3, 45, 70, 90, 8, "f32", True),
    ("forward_four_rows_four_waves", 41, 30, 66, 75, 4, "f32", True),
    ("forward_four_rows_bf16", 41, 30, 66, 131, 4, "bf16", False),
    ("forward_slices_of_64", 110, 30, 66, 41, 4, "f32", True),
    ("forward_slices_of_128", 110, 29, 66, 102, 4, "f32", True),
    ("forward_slices_of_128_bf16", 110, 31, 70, 103, 4, "bf16", False),
    # the same forms beyond H = 512, up to 128 columns, and on few keys
    ("forward_four_rows_wide_h", 41, 90, 66, 530, 4, "f32", True),
    ("forward_slices_of_64_wide_h", 60, 220, 33, 517, 4, "f32", True),
    ("forward_slices_of_128_wide_h_bf16", 90, 76, 50, 590, 4, "bf16", False),
    ("forward_full_slices_of_64", 140, 30, 66, 41, 4, "f32", True),
    ("forward_full_slices_of_128", 140, 29, 66, 243, 4, "f32", True),
    ("forward_full_slices_of_128_bf16", 140, 31, 70, 241, 4, "bf16", False),
    ("forward_full_slices_of_256", 50, 53, 40, 1001, 4, "f32", True),
    # few keys on more than a round of blocks: one key, as many as lane groups, past 16 with three slices of h and with up to 128 columns;
    # many blocks with the keys of the row mode
    ("forward_few_keys_many_blocks", 300, 9, 1, 33, 4, "f32", False),
    ("forward_few_keys_many_blocks_16", 256, 15, 16, 130, 68, "f32", True),
    ("forward_few_keys_many_blocks_bf16", 180, 23, 9, 645, 8, "bf16", False),
    ("forward_17_keys_many_blocks_wide_h", 256, 11, 17, 600, 36, "f32", True),
    ("forward_32_keys_many_blocks", 200, 46, 32, 127, 4, "f32", True),
    ("forward_33_keys_past_four_rounds", 230, 66, 33, 129, 12, "f32", True),
    ("forward_49_keys_many_blocks", 120, 47, 49, 258, 132, "f32", True),
    ("forward_49_keys_many_blocks_bf16", 190, 57, 64, 300, 260, "bf16", False),
    # beyond H = 512: four rows in eight waves at their last grid, four rows in four waves next to it on short key axes, then eight
    # rows in eight waves, and four rows in four waves again where slices of 256 columns waste lanes
    ("forward_wide_four_rows_eight_waves", 36, 61, 70, 530, 4, "f32", True),
    ("forward_wide_four_rows_eight_waves_bf16", 26, 62, 40, 643, 36, "bf16", False),
    ("forward_wide_four_rows_four_waves", 37, 61, 60, 530, 4, "f32", False),
    ("forward_wide_four_rows_four_waves_bf16", 37, 61, 60, 530, 68, "bf16", False),
    ("forward_wide_four_rows_four_waves_700", 27, 61, 40, 700, 4, "f32", True),
    ("forward_wide_eight_rows", 45, 61, 70, 516, 132, "f32", True),
    ("forward_wide_eight_rows_bf16", 27, 61, 40, 767, 4, "bf16", False),
    ("forward_wide_four_rows_again", 64, 61, 70, 637, 4, "f32", False),
    ("forward_three_slices_512_blocks", 128, 25, 27, 516, 12, "f32", True),
    ("forward_three_slices_past_512_blocks", 129, 25, 27, 516, 12, "f32", False),
    ("forward_row_mode_three_slices", 9, 21, 32, 513, 8, "f32", True),
    ("forward_row_mode_three_slices_bf16", 9, 5, 20, 767, 516, "bf16", False),
    ("forward_few_keys_full_grid", 180, 22, 13, 600, 4, "f32", True),
    ("forward_few_keys", 9, 5, 11, 662, 8, "f32", True),
    # context with a share of the keys per wave: one, two and four columns per lane, one to four groups of columns with a short
    # last one, shares without keys (few valid keys), four and eight waves, blocks of four and eight rows
    ("context_shares_4_columns", 140, 30, 66, 44, 4, "f32", False),
    ("context_shares_60_columns_bf16", 41, 30, 70, 44, 60, "bf16", False),
    ("context_shares_64_columns", 3, 45, 70, 90, 64, "f32", False),
    ("context_shares_68_columns", 140, 29, 67, 36, 68, "f32", False),
    ("context_shares_128_columns_bf16", 3, 45, 70, 90, 128, "bf16", False),
    ("context_shares_132_columns", 41, 31, 131, 52, 132, "f32", False),
    ("context_shares_256_columns", 140, 30, 66, 20, 256, "f32", False),
    ("context_shares_260_columns", 3, 9, 300, 40, 260, "f32", False),
    ("context_shares_512_columns_bf16", 41, 30, 66, 40, 512, "bf16", False),
    ("context_few_keys_104_columns", 180, 20, 11, 662, 104, "f32", False),
    ("context_36_keys_of_wide_h", 9, 13, 36, 601, 300, "f32", False),
    ("context_shares_37_keys", 9, 13, 37, 601, 300, "f32", False),
    ("context_no_shares_516_columns", 41, 30, 66, 40, 516, "f32", False),
    ("context_shares_516_columns_eight_waves", 3, 45, 70, 36, 516, "f32", False),
    ("context_shares_row_mode_1000_columns", 5, 21, 50, 512, 1000, "f32", False),
    ("context_shares_wide_h", 50, 53, 40, 1001, 772, "bf16", False),
    ("forward_spread_small_batch", 9, 150, 67, 36, 8, "f32", False),
    ("forward_row_mode_odd_h", 3, 21, 20, 250, 8, "f32", True),
    ("forward_row_mode_odd_h_bf16", 3, 21, 20, 511, 8, "bf16", False),
    ("forward_eight_waves_odd_h", 70, 61, 66, 777, 4, "f32", False),
    # pre-kernel in parts (few blocks, more than 128 keys): parts of 64 keys with a short last one, masked parts, one and two
    # rounds over the value columns, rows and columns that are no multiples of the tiles, few rows for the four waves of dV
    ("pre_parts_one_key_in_the_last", 2, 45, 129, 40, 24, "f32", False),
    ("pre_parts_two_rounds", 3, 33, 200, 24, 708, "f32", False),
    ("pre_parts_full_round", 2, 17, 256, 24, 512, "f32", False),
    ("pre_parts_few_rows_bf16", 4, 3, 137, 24, 68, "bf16", False),
    ("pre_parts_two_rounds_bf16", 2, 70, 190, 24, 1024, "bf16", False),
    ("pre_parts_keys_past_384", 1, 90, 470, 24, 40, "f32", False),
    # without parts, on split operands: five to twelve key tiles of 32 for the eight waves, the last one full or short; value rows of less than a
    # chunk of 32 columns, two and a bit, four and a bit; at most 16 rows
    ("pre_split_129_keys", 101, 32, 129, 8, 4, "f32", False),
    ("pre_split_255_keys", 51, 65, 255, 8, 68, "f32", False),
    ("pre_split_319_keys_bf16", 40, 97, 319, 8, 132, "bf16", False),
    ("pre_split_384_keys", 60, 33, 384, 8, 60, "f32", False),
    ("pre_split_333_keys_bf16", 102, 17, 333, 8, 64, "bf16", False),
    ("pre_split_333_keys_76_columns_bf16", 102, 17, 333, 8, 76, "bf16", False),
    ("pre_split_384_keys_100_columns", 60, 33, 384, 8, 100, "f32", False),
    ("pre_split_16_rows_300_keys", 101, 16, 300, 8, 44, "f32", False),
    ("pre_split_15_rows_317_keys_bf16", 105, 15, 317, 8, 132, "bf16", False),
    ("pre_split_390_keys", 60, 50, 390, 8, 44, "f32", False),
    # pre-kernel on split operands: 17 to 64, 65 to 128 and more keys (up to two key tiles of 32 per wave, and none); rows that are no multiple
    # of 32 and of the 64 of a dV step, one step and several; value rows of less than a chunk of 32 columns, exactly one, part of a second
    # one, an odd number of them, more chunks than waves, more columns than a dV block; key panels of 64 with one key in the last; and
    # the fewest blocks that take it, next to one that does not
    ("pre_split_17_keys", 130, 17, 17, 8, 4, "f32", False),
    ("pre_split_64_keys_36_columns", 130, 33, 64, 8, 36, "f32", False),
    ("pre_split_64_keys_260_columns_bf16", 130, 65, 64, 8, 260, "bf16", False),
    ("pre_split_33_keys_544_columns", 64, 32, 33, 8, 544, "f32", False),
    ("pre_not_split_63_blocks", 63, 32, 33, 8, 544, "f32", False),
    ("pre_split_1060_columns_bf16", 40, 64, 40, 8, 1060, "bf16", False),
    ("pre_split_65_keys_32_columns", 130, 64, 65, 8, 32, "f32", False),
    ("pre_split_128_keys_100_columns", 70, 129, 128, 8, 100, "f32", False),
    ("pre_split_97_keys_96_columns_bf16", 70, 31, 97, 8, 96, "bf16", False),
    ("pre_split_100_keys_384_columns", 64, 60, 100, 8, 384, "f32", False),
    ("pre_split_100_keys_388_columns", 64, 60, 100, 8, 388, "f32", False),
    ("pre_split_128_keys_512_columns", 64, 33, 128, 8, 512, "f32", False),
    ("pre_split_444_columns", 128, 33, 100, 8, 444, "f32", False),
    ("pre_not_split_448_columns", 128, 33, 100, 8, 448, "f32", False),
    ("pre_not_split_512_columns", 128, 33, 65, 8, 512, "f32", False),
    ("pre_split_516_columns", 128, 33, 65, 8, 516, "f32", False),
    ("pre_split_255_blocks", 255, 17, 128, 8, 512, "f32", False),
    ("pre_split_129_keys_516_columns", 201, 17, 129, 8, 516, "f32", False),
    ("pre_split_257_keys_36_columns", 50, 70, 257, 8, 36, "f32", False),
    ("pre_split_512_keys_64_columns_bf16", 51, 64, 512, 8, 64, "bf16", False),
    ("pre_not_split_513_keys", 51, 64, 513, 8, 64, "f32", False),
    # more than 512 keys, fp32 products in blocks of 16 rows: dV in panels of 64 keys (800 panels, or up to 16 rows) and in blocks of 16 keys
    # (fewer panels, or P rows that are no whole 16 bytes), remainders of the rows, value rows that are no whole 32 columns and more than
    # 1024; and in parts up to 100 blocks of 32 rows, 200 of wide rows
    ("pre_long_panels_44_columns_bf16", 101, 18, 516, 8, 44, "bf16", False),
    ("pre_long_panels_one_key_group_short", 134, 17, 580, 8, 4, "f32", False),
    ("pre_long_panels_9_rows", 101, 9, 520, 8, 44, "f32", False),
    ("pre_long_panels_1028_columns", 21, 17, 516, 8, 1028, "f32", False),
    ("pre_long_16_keys_132_columns", 101, 33, 513, 8, 132, "f32", False),
    ("pre_long_few_panels_132_columns_bf16", 51, 65, 516, 8, 132, "bf16", False),
    ("pre_long_1028_columns_bf16", 3, 20, 515, 8, 1028, "bf16", False),
    ("pre_long_parts_100_blocks", 50, 64, 516, 8, 40, "f32", False),
    ("pre_long_parts_200_blocks_bf16", 100, 33, 513, 8, 388, "bf16", False),
    # short runs of products summed on their own: the most blocks that do it, narrow and wide value rows, and one more
    ("pre_apart_100_blocks", 50, 33, 129, 8, 380, "f32", False),
    ("pre_apart_200_blocks_bf16", 100, 33, 257, 8, 388, "bf16", False),
    ("pre_apart_one_row", 51, 1, 512, 8, 36, "f32", False),
    ("pre_not_apart_101_blocks", 101, 17, 129, 8, 380, "f32", False),
    # one block per CU: the fewest keys, columns, blocks and rows per block that take it, and one key, four columns, one sample and one row less;
    # several key tiles per wave
    ("pre_alone_193_keys_512_columns", 128, 48, 193, 4, 512, "f32", False),
    ("pre_not_alone_192_keys", 128, 48, 192, 4, 512, "f32", False),
    ("pre_not_alone_508_columns", 128, 48, 193, 4, 508, "f32", False),
    ("pre_not_alone_254_blocks", 127, 48, 193, 4, 512, "f32", False),
    ("pre_not_alone_47_rows", 128, 47, 193, 4, 512, "f32", False),
    ("pre_alone_512_keys_548_columns", 65, 125, 512, 4, 548, "f32", False),
    # whole backward in one launch: one tile, remainders of the tiles, one row, one key, three tiles, all sixteen with two per wave,
    # slices of 16 to 64 columns, several pieces of columns of each width, entries that need the exponential of the sum
    ("small_one_tile", 4, 6, 7, 16, 16, "f32", True),
    ("small_one_row_one_key", 3, 1, 1, 20, 4, "f32", False),
    ("small_full", 2, 64, 64, 40, 96, "f32", True),
    ("small_three_row_tiles", 3, 47, 16, 33, 68, "f32", False),
    ("small_three_key_tiles_bf16", 3, 15, 33, 100, 132, "bf16", False),
    ("small_pieces_of_256", 2, 16, 13, 64, 600, "f32", False),
    ("small_pieces_of_128", 2, 17, 32, 70, 260, "f32", False),
    ("small_slices_of_64", 10, 50, 60, 128, 64, "f32", True),
    ("small_many_blocks_bf16", 25, 30, 29, 96, 100, "bf16", False),
    ("forward_h_4", 2, 9, 13, 4, 4, "f32", False),
    ("forward_h_5", 2, 9, 13, 5, 4, "f32", False),
    ("forward_h_7_bf16", 2, 9, 70, 7, 4, "bf16", False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_launch_form(case):
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import harness
    name, B, Tq, Tk, H, Dv, dt, big = case
    print("launch form", case, flush=True)
    wl = Workload(name, B, Tq, Tk, H, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    inputs = make_inputs(wl, seed=313 + len(name))
    if B > 2:
        inputs["key_len"][1] = 0                              # a sample without a valid key among the others
    if big:
        inputs["Qp"][0, Tq // 2, : H // 2] = 60.0
        inputs["Kp"][0, 0, : H // 2] = -59.5
        inputs["Kp"][B - 1, Tk - 1, H // 3] = 45.0
        inputs["key_len"][B - 1] = Tk
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    db.fwd()
    db.bwd()
    got = db.results()
    assert db.check_guards() == []
    assert_parity(got, oracle_outputs(inputs, workers=1), inputs, dt, name)
    first = {k: v.copy() for k, v in got.items()}
    db.fwd()
    db.bwd()
    again = db.results()
    for k in first:
        assert np.array_equal(first[k], again[k]), (name, k, "not reproducible")


PARTS = [
    # B, Tq, Tk, Dv, dtype, whether the pre-kernel runs in parts: up to 50 blocks of 32 rows where the other form would be split operands, up to
    # 100 or 200 where it would be fp32 products
    (50, 32, 129, 8, "f32", True), (51, 32, 129, 8, "f32", False), (50, 1, 512, 1024, "bf16", True), (51, 1, 512, 1024, "bf16", False),
    (100, 32, 513, 380, "f32", True), (101, 32, 513, 380, "f32", False), (200, 3, 516, 384, "bf16", True), (201, 3, 516, 384, "bf16", False),
    (3, 40, 600, 1028, "f32", False), (40, 20, 128, 8, "f32", False),
]


@pytest.mark.parametrize("case", PARTS, ids=["_".join(map(str, c[:5])) for c in PARTS])
def test_which_launches_run_in_parts(case):
    """The launch that finishes the parts is there exactly where the rule says (a limit drawn for split operands had also held where there are
    none: up to twice the time past 512 keys)."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb, harness
    B, Tq, Tk, Dv, dt, parts = case
    print("parts", case, flush=True)
    wl = Workload("parts", B, Tq, Tk, 100, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    db = harness.DeviceBatch(wl, make_inputs(wl, seed=3), guard_bytes=4096)
    db.fwd()
    eb.echo_attn_profile_enable(True)
    try:
        eb.echo_attn_profile_read()
        db.bwd()
        torch.cuda.synchronize()
        names = eb.echo_attn_profile_read()
    finally:
        eb.echo_attn_profile_enable(False)
    assert "bwd_pre" in names and ("ds_finish" in names) == parts, names


LARGE_ROWS = [
    # name, B, Tq, Tk, H, Dv, dtype, queries beyond the factor limit as (sample, row): recomputation with up to 25 rows per lane in
    # several passes, one of them on the factor path and one not, with a first step that does not deal its keys evenly to the waves
    ("first_pass", 236, 201, 13, 99, 4, "f32", [(0, 7)]),
    ("last_pass", 236, 201, 21, 99, 4, "f32", [(3, 190)]),
    ("middle_pass_bf16", 331, 405, 9, 99, 4, "bf16", [(0, 200), (5, 150)]),
]


@pytest.mark.parametrize("case", LARGE_ROWS, ids=[c[0] for c in LARGE_ROWS])
def test_passes_with_and_without_large_entries(case):
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import harness
    name, B, Tq, Tk, H, Dv, dt, rows = case
    print("large rows", case, flush=True)
    wl = Workload(name, B, Tq, Tk, H, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    inputs = make_inputs(wl, seed=71 + len(name))
    for b, row in rows:
        put_rows(inputs, dt, "Qp", (b, row, slice(None, None, 2)), 40.5)
        put_rows(inputs, dt, "Kp", (b, slice(None, None, 3), slice(None, None, 2)), -39.75)    # (still within the limit)
        inputs["key_len"][b] = Tk
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    db.fwd()
    db.bwd()
    got = db.results()
    assert db.check_guards() == []
    assert_parity(got, oracle_outputs(inputs, workers=1), inputs, dt, name)
    db.bwd()
    again = db.results()
    for k in got:
        assert np.array_equal(got[k], again[k]), (name, k, "not reproducible")


STEPS = [
    # name, B, Tk, H, Dv, dtype: one decoder step and its query gradient, the sample's block at the edges of its batches
    # (64 rows, 512 columns): one batch of each matrix, one row and one column more, three batches, rows of one to three
    # elements, tails of one to three columns, both storage types
    ("one_batch_full", 3, 64, 512, 512, "f32"),
    ("one_batch_bf16_tail", 70, 33, 301, 260, "bf16"),
    ("one_more_row", 3, 65, 512, 512, "f32"),
    ("one_more_column", 3, 20, 513, 516, "f32"),
    ("three_batches_of_rows_and_columns", 2, 150, 1030, 1100, "f32"),
    ("many_rows_bf16", 2, 331, 77, 40, "bf16"),
    ("h_1", 3, 70, 1, 4, "f32"),
    ("h_2_bf16", 3, 20, 2, 8, "bf16"),
    ("h_3", 3, 130, 3, 516, "f32"),
    ("h_4", 3, 66, 4, 4, "f32"),
    # forward in blocks of eight waves: the last count of keys that takes it and the first that does not, by width, number of
    # samples and type; columns and value columns that are no multiples of its 256 and 512
    ("rows_16_keys", 5, 16, 75, 620, "f32"),
    ("rows_not_17_keys", 5, 17, 75, 620, "bf16"),
    ("rows_6_keys_wide", 5, 6, 1000, 1004, "f32"),
    ("rows_not_7_keys_wide", 5, 7, 1000, 1004, "f32"),
    ("rows_4_keys_of_odd_h", 129, 4, 587, 20, "f32"),
    ("rows_not_5_keys_of_odd_h", 129, 5, 587, 20, "bf16"),
    ("rows_10_keys_past_128_samples", 129, 10, 516, 36, "bf16"),
    ("rows_32_keys_past_256_samples", 257, 32, 131, 880, "f32"),
    ("rows_17_keys_past_256_samples_bf16", 257, 17, 428, 516, "bf16"),
    ("rows_one_key", 300, 1, 514, 4, "f32"),
    ("rows_h_3_100_keys", 260, 100, 3, 8, "f32"),
    # query gradient in blocks per 64 columns: one key, one and several batches of 32 keys, a last slice of one column, the limits
    # on keys, blocks and value bytes
    ("slices_one_key", 7, 1, 65, 4, "f32"),
    ("slices_300_keys", 4, 300, 700, 40, "bf16"),
    ("slices_not_301_keys", 4, 301, 512, 40, "f32"),
    ("slices_any_keys_32_blocks", 2, 410, 1024, 1024, "f32"),
    ("slices_16_mb", 100, 163, 128, 128, "f32"),
    ("slices_not_past_16_mb", 100, 164, 128, 128, "f32"),
    ("slices_26_mb_of_wide_rows", 20, 100, 640, 644, "bf16"),
    ("slices_900_blocks", 100, 32, 520, 20, "f32"),
    ("slices_not_901_blocks", 101, 5, 520, 20, "bf16"),
    ("slices_not_601_blocks_of_one_batch", 121, 9, 301, 20, "f32"),
    ("slices_1500_blocks", 300, 33, 301, 20, "f32"),
    ("slices_one_past_256_samples", 257, 70, 64, 24, "bf16"),
]


@pytest.mark.parametrize("case", STEPS, ids=[c[0] for c in STEPS])
def test_step_of_one_query(case):
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb, harness
    name, B, Tk, H, Dv, dt = case
    print("step", case, flush=True)
    wl = Workload(name, B, 1, Tk, H, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    inputs = make_inputs(wl, seed=99 + len(name))
    inputs["key_len"][0] = Tk
    if B > 2:
        inputs["key_len"][1] = 0
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    ds = torch.full((eb.echo_attn_steps_ds_bytes(db.desc),), 0xFF, dtype=torch.uint8, device=db.device)
    st = torch.cuda.current_stream(db.device)
    eb.check(eb.echo_attn_step_fwd(db.desc, db.Qp, db.Kp, db.V, db.v, db.key_len, db.context, db.P, stream=st))
    eb.check(eb.echo_attn_step_bwd_query(db.desc, 0, 1, db.dC, db.P, db.Qp, db.Kp, db.V, db.v, db.key_len, db.dQp, ds, stream=st))
    eb.check(eb.echo_attn_steps_bwd_keys(db.desc, db.dC, db.P, db.Qp, db.Kp, db.v, db.key_len, ds, db.dKp, db.dV, db.dv, db.ws,
                                         stream=st))
    got = db.results()
    assert db.check_guards() == []
    assert_parity(got, oracle_outputs(inputs, workers=1), inputs, dt, name)


KEYS_ALONE = [
    # B, Tq, Tk, Dv, dtype: dV of the keys' call on more than 50 blocks and past 128 keys: up to 12 rows in fp32, in panels of 64 keys or, where
    # P rows are no whole 16 bytes, in blocks of 16; more rows on split operands
    (60, 12, 132, 260, "f32"), (60, 13, 132, 260, "f32"), (60, 12, 131, 36, "bf16"), (60, 13, 131, 36, "bf16"), (60, 1, 512, 1028, "f32"),
    (60, 5, 129, 4, "f32"), (60, 7, 513, 68, "f32"),
]


@pytest.mark.parametrize("case", KEYS_ALONE, ids=["_".join(map(str, c)) for c in KEYS_ALONE])
def test_values_gradient_of_few_rows(case):
    """dV = P^T dC over Tq terms: a product and at most Tq additions of fp32, and the two roundings that split operands add, of the terms'
    magnitudes."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb, harness
    B, Tq, Tk, Dv, dt = case
    print("keys alone", case, flush=True)
    wl = Workload("keys", B, Tq, Tk, 8, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    inputs = make_inputs(wl, seed=41)
    inputs["key_len"][:3] = (0, Tk, 1)
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    db.fwd()
    ds = torch.zeros(eb.echo_attn_steps_ds_bytes(db.desc), dtype=torch.uint8, device=db.device)
    eb.check(eb.echo_attn_steps_bwd_keys(db.desc, db.dC, db.P, db.Qp, db.Kp, db.v, db.key_len, ds, db.dKp, db.dV, db.dv, db.ws,
                                         stream=torch.cuda.current_stream(db.device)))
    torch.cuda.synchronize()
    assert db.check_guards() == []
    P, dC, dV = (x.cpu().numpy().astype(np.float64) for x in (db.P, db.dC, db.dV))
    for b in range(B):
        L = int(inputs["key_len"][b])
        assert (dV[b, L:] == 0).all(), b
        bound = (Tq + 3) * 2.0 ** -24 * (np.abs(P[b, :, :L]).T @ np.abs(dC[b])) + 1e-44
        assert (np.abs(dV[b, :L] - P[b, :, :L].T @ dC[b]) <= bound).all(), b


ORDERS = [
    # name, B, Tq, Tk, H, samples whose blocks are among the first 256 (0: more than 512 blocks): slices of 64 columns in one round; more
    # than a round of slices of 16 where slices of 64 would be one; every tanh twice in independent blocks; parts of a round; an odd
    # number of samples in one round less a block
    ("one_round", 64, 50, 50, 512, 32),
    ("narrow_slices_past_a_round", 28, 80, 80, 300, 0),
    ("split", 5, 200, 200, 76, 0),
    ("rows_of_25_one_round", 73, 72, 29, 320, 51),
    ("rows_of_25_past_a_round", 140, 72, 40, 320, 0),
    ("part_of_a_round", 41, 35, 28, 512, 32),
    ("rows_of_25_part_of_a_round", 31, 128, 166, 816, 19),
    ("one_alone", 73, 50, 30, 448, 37),
]


@pytest.mark.parametrize("case", ORDERS, ids=[c[0] for c in ORDERS])
def test_order_of_the_samples_in_the_recompute_grid(case):
    """Heaviest sample first; in a grid that runs all at once, where a block's compute unit also gets the block 256 later, heavy samples
    meet light ones and the heaviest meet nobody.  The order is the run of `sample | keys << 16` words that the backward leaves in its
    workspace."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import harness
    name, B, Tq, Tk, H, first = case
    print("order", case, flush=True)
    wl = Workload(name, B, Tq, Tk, H, 4, "f32", 0.5, 1, Tk, False)
    inputs = make_inputs(wl, seed=17)
    inputs["key_len"] = np.random.default_rng(17).integers(1, Tk + 1, B).astype(np.int32)
    db = harness.DeviceBatch(wl, inputs)
    db.poison_outputs()
    db.fwd()
    db.bwd()
    torch.cuda.synchronize()
    words = db.ws.view(torch.int32).cpu().numpy()
    is_entry = np.zeros(words.size, dtype=bool)
    for b, L in enumerate(inputs["key_len"]):
        is_entry |= words == (b | int(L) << 16)
    runs = [k for k in np.flatnonzero(is_entry) if is_entry[k:k + B].all() and len(set(words[k:k + B] & 0xffff)) == B]
    assert len(runs) == 1, runs
    lengths = words[runs[0]:runs[0] + B] >> 16
    if not first:
        assert (np.diff(lengths) <= 0).all(), lengths
        return
    both, light = lengths[:B - first], lengths[first:]               # samples that meet
    alone = lengths[B - first:first]
    assert (np.diff(both) <= 0).all() and (np.diff(alone) <= 0).all() and (np.diff(light) >= 0).all(), lengths
    if len(alone) > 1:
        assert alone.min() >= both.max(initial=0), lengths
    assert lengths[:first].min() >= light.max(initial=0), lengths


ACCUMULATE = [
    # name, B, Tq, Tk, H, Dv, dtype[, queries per pass]: the accumulating call through every tanh twice in independent blocks (several groups of keys, the
    # last ones masked; behind the pre-kernel in parts), the whole backward in one launch, slices of 16 and 32 columns
    ("split", 3, 61, 83, 90, 8, "f32"),
    ("split_bf16", 2, 37, 261, 100, 8, "bf16"),
    ("split_pre_kernel_in_parts", 2, 33, 150, 64, 24, "f32"),
    ("small", 10, 24, 30, 64, 32, "f32"),
    ("slices_of_16", 25, 50, 21, 130, 8, "f32"),
    ("slices_of_32", 34, 45, 9, 470, 8, "f32"),
    ("rows_of_25", 182, 72, 29, 128, 8, "f32"),
    ("rows_of_25_one_group", 202, 130, 13, 126, 4, "bf16"),
    # more than one pass over the queries, large entries (in the first and the last sample, a query and a key each)
    ("rows_of_25_two_passes", 236, 201, 13, 99, 4, "f32", 101),
    ("rows_of_25_three_passes_large", 331, 405, 9, 99, 4, "f32", 135),
    ("rows_of_25_large_bf16", 182, 72, 29, 128, 8, "bf16"),
]


@pytest.mark.parametrize("case", ACCUMULATE, ids=[c[0] for c in ACCUMULATE])
def test_accumulating_backward(case):
    """dKp, dV and dv are added to what the buffers hold, in one rounding of the sum; where a masked key adds nothing the buffer
    stays as it is, bit for bit.  dQp is overwritten."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb, harness
    name, B, Tq, Tk, H, Dv, dt, *per_pass = case
    print("accumulate", case, flush=True)
    wl = Workload(name, B, Tq, Tk, H, Dv, dt, 0.5, 1, Tk, dt == "bf16")
    inputs = make_inputs(wl, seed=41 + len(name))
    inputs["key_len"][0] = Tk // 3                        # whole groups of masked keys
    inputs["key_len"][1] = 0
    if "large" in name:
        inputs["key_len"][B - 1] = Tk
        for b, row, key in ((0, 5, 0), (B - 1, Tq - 3, Tk - 2)):
            put_rows(inputs, dt, "Qp", (b, row, slice(None, None, 2)), 44.0)
            put_rows(inputs, dt, "Kp", (b, key, slice(None, None, 3)), -43.5)
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    db.fwd()
    db.bwd()
    alone = db.results()
    if "large" in name:
        assert_parity(alone, oracle_outputs(inputs, workers=1), inputs, dt, name)
    # what the passes over the queries add to dKp one after the other: dS of the other passes' queries zero with their dC
    parts = []
    for first in range(0, Tq, per_pass[0]) if per_pass else ():
        whole = db.dC.clone()
        db.dC[:, :first] = 0
        db.dC[:, first + per_pass[0]:] = 0
        db.bwd()
        parts.append(np.abs(db.results()["dKp"]))
        db.dC.copy_(whole)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    held = {}
    for k in ("dKp", "dV", "dv"):
        t = getattr(db, k)
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
        held[k] = t.cpu().numpy()
    db.dQp.fill_(float("nan"))
    eb.check(eb.echo_attn_bwd_accumulate(db.desc, db.dC, db.P, db.Qp, db.Kp, db.V, db.v, db.key_len, db.dQp, db.dKp, db.dV, db.dv,
                                         db.ws, stream=torch.cuda.current_stream(db.device)))
    got = db.results()
    assert db.check_guards() == []
    assert np.array_equal(got["dQp"], alone["dQp"])
    for k, base in held.items():
        # a few roundings of the larger of sum and parts: over n passes n of sums of up to all parts, and n - 1 in `alone`
        size = np.abs(base) + (sum(parts) if parts and k == "dKp" else np.abs(alone[k]))
        roundings = max(4, 2 * len(parts))
        assert (np.abs(got[k] - (base.astype(np.float64) + alone[k])) <= roundings * 2.0 ** -24 * size + 1e-30).all(), k
    for b, L in enumerate(np.clip(inputs["key_len"], 0, Tk)):
        assert np.array_equal(got["dKp"][b, L:], held["dKp"][b, L:]) and np.array_equal(got["dV"][b, L:], held["dV"][b, L:])


@pytest.mark.parametrize("lengths", ["equal", "two", "top_bits_equal", "any"])
@pytest.mark.parametrize("B", [65, 128, 129, 256])
def test_forward_order_of_the_samples(B, lengths):
    """Every sample has to come up once whatever the lengths tie in: all equal, two of them, all with the same leading bits, all different
    ones; two lengths per lane (up to 128 samples) and four."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import harness
    Tq, Tk, H = 8 * (705 // B) + 8, 66, 228                    # (more than 700 blocks of eight rows, 66 x 228 > 15000)
    print("order of the samples", B, lengths, flush=True)
    wl = Workload(f"order_{B}_{lengths}", B, Tq, Tk, H, 4, "f32", 0.5, 1, Tk, False)
    inputs = make_inputs(wl, seed=B)
    rng = np.random.default_rng(B)
    inputs["key_len"][:] = {"equal": np.full(B, 7), "two": rng.choice([0, Tk], B), "top_bits_equal": rng.integers(64, 67, B),
                            "any": rng.integers(0, Tk + 1, B)}[lengths]
    db = harness.DeviceBatch(wl, inputs, guard_bytes=4096)
    db.poison_outputs()
    db.fwd()
    db.bwd()
    got = db.results()
    assert db.check_guards() == []
    assert_parity(got, oracle_outputs(inputs), inputs, "f32", wl.name)
