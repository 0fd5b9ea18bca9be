"""Which kernels a call of given sizes takes, on the CPU (the rules' measured reasons stand in
csrc/sort_choice.h, csrc/ingest_choice.h and csrc/join_choice.h)."""
import pytest

from kernel_choice import MERGE, PART, RADIX, RANK, SPLIT, plain_copy, choice, commit_apart, least_fences, ranges_of_viewers


@pytest.mark.parametrize("sizes,max_keys,want", [
    ([5_000], 0, RANK), ([10_240], 0, RANK), ([10_241], 0, SPLIT), ([500] * 80, 500, RANK),
    ([500] * 81, 500, PART), ([5_000] * 4, 5_000, PART), ([100] * 90, 100, PART),
    ([5_000] * 64, 5_000, PART), ([5_000] * 64, 8_192, PART), ([5_000] * 64, 8_193, SPLIT),
    ([30_000] * 64, 30_000, SPLIT), ([254 * 640] * 20, 254 * 640, SPLIT), ([100_000], 0, SPLIT),
    ([254 * 640 + 1], 0, SPLIT), ([400_000] * 3, 400_000, RADIX), ([400_000], 400_000, SPLIT),
    ([1 << 19], 0, SPLIT), ([(1 << 19) + 1], 0, MERGE), ([5_000] * 105, 0, MERGE),
    ([9_000] * 300, 0, RADIX), ([1_000] * 20_000, 1_000, PART)])
def test_methods(sizes, max_keys, want):
    assert choice(sizes, max_keys) == want


@pytest.mark.parametrize("longest", [160_000, 300_000, 500_000])
def test_a_call_without_a_bound_may_hold_one_long_viewer(longest):
    """One viewer of nearly all records among 1,000: 158 us (300,000) to 257 (500,000) in one launch, where
    merge takes 116 to 126 and two launches 64 to 80. With a bound on its viewers, or lists so short
    that merge pays more for their number, the one launch is the faster one."""
    sizes = [longest] + [20] * 1_000
    assert choice(sizes) == SPLIT
    assert choice([5_000] * 64) == SPLIT and choice([5_000] * 64, 5_000) == PART
    assert choice([longest] + [1] * 8_000) == PART
    assert choice([10] * 20_000) == PART


@pytest.mark.parametrize("sizes,want", [
    ([180_000] * 2, SPLIT), ([262_000], SPLIT), ([180_000] * 3, MERGE), ([5_000] * 2_000, RADIX), ([5_000] * 2_700, RADIX),
    ([8_000] * 900, RADIX), ([8_000] * 300, PART), ([5_000] * 500, PART), ([2_000] * 2_000, PART),
    ([1_280] * 40_000, PART), ([1_281] * 40_000, RADIX)])
def test_the_partitions_key_reads_have_a_limit(sizes, want):
    """Past it the other methods are faster, by 2 to 22%; viewers of one part read no key twice."""
    assert choice(sizes, max(sizes)) == want


def test_very_many_very_short_lists():
    """8 records each: 12.3 ms with radix, 17.5 in one launch."""
    assert choice([8] * 1_200_000, 16) == RADIX and choice([16] * 600_000, 16) == RADIX
    assert choice([24] * 600_000, 24) == PART and choice([8] * 100_000, 16) == PART


@pytest.mark.parametrize("n,row,want", [
    (300_000, 128, False), (2_000_000, 128, False), (1_000_000, 256, False), (100_000, 2_048, False),
    (600_000, 1_024, True), (1_000_000, 512, True), (2_000_000, 256, True), (1_500_000, 1_024, True),
    (1 << 21, 16, True)])
def test_batches_of_many_row_bytes_update_the_map_apart(n, row, want):
    """1,500,000 records of 1,024 bytes: 862 us in one launch, 781 in two."""
    assert commit_apart(n, row) == want


@pytest.mark.parametrize("viewers,keys,want", [
    (1, 68_767, 4_096), (1, 5_000_000, 4_096), (100, 20_000, 4_096), (300, 20_000, 4_096),
    (32, 60_000, 4_096), (64, 60_000, 512), (100, 40_000, 512), (100, 60_000, 512)])
def test_short_segments_of_many_long_lists_stage_few_fences(viewers, keys, want):
    """100 viewers of 60,000 keys with 10 candidates each: 10 us with 512 fences, 15.7 with 4,096."""
    assert least_fences(viewers, keys) == want


@pytest.mark.parametrize("n,viewers,want", [
    (40, 16, 48), (8, 3, 9), (16, 100, 100), (256, 64, 256), (256, 12, 252), (256, 100, 0), (256, 17, 255),
    (256, 33, 0), (256, 240, 240), (256, 300, 0), (200, 150, 0), (64, 256, 256)])
def test_ranges_of_small_launches_are_a_multiple_of_the_viewers(n, viewers, want):
    """So that no range of equal viewers holds parts of two: 16 viewers of 160 candidates 8.3 us, 12.0 on
    40 ranges."""
    got = ranges_of_viewers(n, viewers, 256)
    assert got == want and got % viewers == 0 and got <= 256


@pytest.mark.parametrize("rows,stride,width,want", [
    (10_000, 32, 32, False), (10_000, 80, 32, True), (50_000, 80, 32, True), (200_000, 48, 32, False),
    (10_000, 80, 64, False)])
def test_small_outputs_of_short_rows_with_gaps_take_no_pipeline(rows, stride, width, want):
    """10,000 rows of 32 bytes at 80: 5.7 us with it, 5.0 without."""
    assert plain_copy(rows, stride, width) == want
