"""GPU parity of the sort's methods that only the automatic choice takes (ranks by comparison, the
partition in one launch, and in two for long viewers) against the oracle's stable sort: sizes around
a part, the LDS tile and the sample; key distributions that break the sample's estimate; bounds;
malformed offsets. Every case names the method that its sizes are meant to lead to, and asks the rule
itself (kernel_choice) whether they do."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2609_22441_amd as P
import workload as W
from gpu_common import note
from kernel_choice import MERGE, PART, RANK, SPLIT, choice

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHORT, LONG = 1024, 1280     # records per part in calls of at most 2^18 records, and of more
BOUND = 8_192                # the longest list that the partition takes in one launch by its bound
KINDS = ["ids", "few", "equal", "ascending", "descending", "wide", "top"]


def _sort(ko, keys, rows, max_keys=0):
    n = keys.numel()
    ws = torch.full((max(16, P.cc_sort_workspace_bytes(n, ko.numel() - 1)),), 0xEE,
                    dtype=torch.uint8, device=DEV)
    k_out = torch.full((n,), -7, dtype=torch.int64, device=DEV)
    r_out = torch.full(rows.shape, 0xCD, dtype=torch.uint8, device=DEV)
    P.cc_sort_affinity(ko.to(DEV), keys.to(DEV), rows.to(DEV), k_out, r_out, ws, max_keys=max_keys)
    torch.cuda.synchronize()
    return k_out.cpu().numpy(), r_out.cpu().numpy()


def _check(sizes, keys, what, want, row=16, max_keys=0):
    """`want`: the method that the call is meant to take."""
    note(f"sort method {want}: {what}")
    assert choice(sizes, max_keys) == want, what
    sizes = torch.as_tensor(sizes, dtype=torch.int64)
    ko = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(sizes, 0)])
    n = int(ko[-1])
    assert keys.numel() == n
    g = W.gen("cpu", n, 5)
    rows = torch.randint(0, 256, (n, row), generator=g, dtype=torch.int64).to(torch.uint8)
    gk, gr = _sort(ko, keys, rows, max_keys)
    wk, wr = oracle.sort_affinity(ko, keys, rows)
    assert np.array_equal(gk, wk), f"{what}: keys"
    assert np.array_equal(gr, wr), f"{what}: rows"


def _keys(kind, n, seed):
    g = W.gen("cpu", seed, 6)
    if kind == "ids":                            # distinct-ish author ids
        return torch.randint(0, 10_000_000, (n,), generator=g)
    if kind == "few":                            # long runs of equal keys
        return torch.randint(-3, 4, (n,), generator=g)
    if kind == "equal":
        return torch.full((n,), 77, dtype=torch.int64)
    if kind == "ascending":
        return torch.arange(n) * 3 - n
    if kind == "descending":
        return n - torch.arange(n) // 2
    if kind == "wide":                           # the full 64-bit span, extremes repeated
        k = torch.randint(-(1 << 62), 1 << 62, (n,), generator=g) * 2
        k[::97] = -(1 << 63)
        k[1::101] = (1 << 63) - 1
        return k
    if kind == "top":                            # up to the largest key, in few values at the end
        k = (1 << 63) - 1 - torch.randint(0, 50_000, (n,), generator=g)
        k[::5] = (1 << 63) - 1 - torch.randint(0, 40, ((n + 4) // 5,), generator=g)
        return k
    raise ValueError(kind)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 65, 513, SHORT, SHORT + 1, 4097, 9_001, 20_011, 140_003])
def test_one_viewer(n, kind):
    """By the method that one viewer of n records takes: one part, ranks, or two launches."""
    want = PART if n < 128 else RANK if n <= 10_240 else SPLIT
    _check([n], _keys(kind, n, n), f"one viewer, {n} {kind} records", want, row=48 if n < 5000 else 16)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 513, SHORT, SHORT + 1, 1_537, 4097, BOUND])
def test_viewers_cut_into_parts(n, kind):
    """Viewers of up to eight parts in one launch: above the size whose ranks are counted, within the
    bound that keeps them from being split beforehand."""
    sizes = [n, 8_000, 0, 2_999]
    _check(sizes, _keys(kind, sum(sizes), n), f"{n}, 8,000 and 2,999 {kind} records", PART, max_keys=BOUND)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [2 * LONG, 7_777])
def test_viewers_cut_into_long_parts(n, kind):
    """The same above 2^18 records, whose parts are longer."""
    sizes = [777] + [n] * (300_000 // n) + [BOUND]
    assert sum(sizes) > 1 << 18
    _check(sizes, _keys(kind, sum(sizes), n), f"{n} {kind} records each", PART, max_keys=BOUND)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [25 * SHORT, 26 * SHORT + 1, 130_000])
def test_long_viewer_in_one_launch(n, kind):
    """A call without a bound holds one long viewer among short ones: samples just small enough to be
    ranked by counting, just too large for it, and one of 1,270 records."""
    sizes = [n] + [20] * 60
    _check(sizes, _keys(kind, sum(sizes), n), f"{n} {kind} records among short lists", PART)


@pytest.mark.parametrize("bits", [31, 40, 52, 53, 63])
def test_ranks_with_and_without_room_for_the_position(bits):
    """Keys whose span leaves just enough, and just too few, bits for a record's position in one
    word (n = 1,500: 11 bits), in two groups that lanes alternate between."""
    g = W.gen("cpu", bits, 3)
    keys = torch.randint(0, 40, (1_500,), generator=g)
    keys[1::2] += 1 << (bits - 1)
    _check([1_500, 130], torch.cat([keys, _keys("few", 130, 1)]), f"two groups, bit {bits - 1}", RANK)


@pytest.mark.parametrize("want", [RANK, PART, SPLIT])
@pytest.mark.parametrize("row", [16, 32, 80, 128, 16 * 513])
def test_row_widths(row, want):
    n = 2_500 if row < 1000 else 700
    sizes = [n, 0, 300] + {RANK: [], PART: [8_000, 1_500], SPLIT: [9_000, 30_000]}[want]
    _check(sizes, _keys("ids", sum(sizes), row), f"row width {row}", want, row=row,
           max_keys={RANK: 0, PART: BOUND, SPLIT: 30_000}[want])


@pytest.mark.parametrize("longest,want", [(BOUND, PART), (30_000, SPLIT)])
def test_ragged_viewers(longest, want):
    """Viewers that start and end anywhere against the multiples of a part, empty ones included;
    the call is above 2^18 records, so the partition's longer parts are used."""
    g = W.gen("cpu", 8, 3)
    sizes = torch.cat([torch.tensor([0, 1, 1023, 1024, 1025, 1536, 1537, longest, 0, 4096, 4097]),
                       torch.randint(0, min(longest, 9_000), (80,), generator=g), torch.tensor([0, 2, 0])])
    n = int(sizes.sum())
    assert n > 1 << 18
    _check(sizes, _keys("ids", n, 9), f"ragged, up to {longest}", want, max_keys=longest)


def test_more_viewers_than_one_search_round():
    g = W.gen("cpu", 9, 3)
    sizes = torch.randint(0, 12, (1_700,), generator=g)
    sizes[::230] = 3_000
    _check(sizes, _keys("few", int(sizes.sum()), 3), "1,700 viewers", PART)


def test_very_short_lists_without_a_bound():
    """200,000 records in lists of 10 on average, one of 50,000: one launch, above the size up to which
    a call without a bound may otherwise take it."""
    sizes = torch.full((15_000,), 10)
    sizes[7_000] = 50_000
    _check(sizes, _keys("ids", int(sizes.sum()), 3), "15,000 short lists and a long one", PART)


def test_above_the_radix_threshold_with_a_bound():
    """2^20 records and more in viewers that the caller bounds by 2^17 or less."""
    _check([60_000] * 18, _keys("ids", 18 * 60_000, 4), "18 x 60,000", SPLIT, max_keys=60_000)
    _check([3_000] * 400, _keys("ids", 400 * 3_000, 4), "400 x 3,000", PART, max_keys=3_000)


def _sample_positions(n, parts, per=10, most=4096):
    """The kernel's sample: one hashed position per stratum."""
    s = min(most if parts > most // per else max(64, parts * per), n)
    i = np.arange(s, dtype=np.uint64)
    step = np.uint64((n << 12) // s)
    a, b = (i * step) >> np.uint64(12), ((i + np.uint64(1)) * step) >> np.uint64(12)
    h = (i * np.uint64(2654435761)) & np.uint64(0xFFFFFFFF)
    return (a + ((h * (b - a)) >> np.uint64(32))).astype(np.int64)


def _misjudged(n, parts, per, most):
    """Keys whose sampled records all lie outside the band that the others share (with repeats)."""
    g = W.gen("cpu", n, 7)
    keys = 500_000_000 + torch.randint(0, 700, (n,), generator=g)
    at = torch.from_numpy(_sample_positions(n, parts, per, most))
    keys[at] = torch.randint(0, 1_000_000_000, (at.numel(),), generator=g)
    band = (keys >= 500_000_000) & (keys < 500_000_700)
    assert int(band.sum()) > most
    return keys


def _parts(lead, n, part):
    return 1 + (lead + n - 1) // part - lead // part


@pytest.mark.parametrize("lead,n,part,max_keys", [
    ([], BOUND, SHORT, BOUND), ([6_000], 8_000, SHORT, BOUND), ([7_777, 3], 5_000, SHORT, BOUND),
    ([777] + [7_000] * 38, 8_000, LONG, BOUND), ([20] * 60, 30_000, SHORT, 0), ([10] * 9, 120_000, SHORT, 0)])
def test_part_that_the_sample_misjudged(lead, n, part, max_keys):
    """One part holds far more records than LDS does and is sorted through the workspace; samples of 80
    to 1,190 records."""
    at = sum(lead)
    rest = [3_000] if max_keys else [10] * 9
    keys = torch.cat([_keys("ids", at, 1), _misjudged(n, _parts(at, n, part), 10, 4_096),
                      _keys("few", sum(rest), 2)])
    assert (len(keys) > 1 << 18) == (part == LONG)
    _check(lead + [n] + rest, keys, f"misjudged part, {n} after {at}", PART, max_keys=max_keys)


@pytest.mark.parametrize("max_keys", [1, 1024, 6000])
def test_viewers_above_the_bound_are_copied_through(max_keys):
    sizes = [5000, 20_000, 300, 0, 6001, 1]
    ko = torch.tensor([0] + np.cumsum(sizes).tolist(), dtype=torch.int64)
    n = int(ko[-1])
    keys = _keys("few", n, max_keys)
    rows = torch.arange(n, dtype=torch.int64).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    note(f"sort: bound {max_keys}")
    assert choice(sizes, max_keys) == (RANK if max_keys == 1 else PART)
    gk, gr = _sort(ko, keys, rows, max_keys)
    wk, wr = oracle.sort_affinity(ko, keys, rows)
    for v, size in enumerate(sizes):
        sl = slice(int(ko[v]), int(ko[v + 1]))
        want = (keys.numpy()[sl], rows.numpy()[sl]) if size > max_keys else (wk[sl], wr[sl])
        assert np.array_equal(gk[sl], want[0]), f"viewer {v} ({size}): keys"
        assert np.array_equal(gr[sl], want[1]), f"viewer {v} ({size}): rows"


def _check_inside(off, n, max_keys, want, keys=None, fill=0xEE):
    """The output for offsets that break the rules is unspecified, but the bytes around the buffers stay
    as they were and every row written is one of the call's rows. Returns the number of those."""
    assert choice([n] + [0] * (len(off) - 2), max_keys) == want
    pad = 4_096
    keys = _keys("ids", n, 2) if keys is None else keys
    rows = torch.arange(n).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    k_all = torch.full((n + 2 * pad,), -7, dtype=torch.int64, device=DEV)
    r_all = torch.full((n + 2 * pad, 16), 0xCD, dtype=torch.uint8, device=DEV)
    size = P.cc_sort_workspace_bytes(n, len(off) - 1)
    ws = torch.full((size + pad,), fill, dtype=torch.uint8, device=DEV)
    P.cc_sort_affinity(torch.tensor(off).to(DEV), keys.to(DEV), rows.to(DEV), k_all[pad:pad + n],
                       r_all[pad:pad + n], ws[:size], max_keys=max_keys)
    torch.cuda.synchronize()
    assert bool((k_all[:pad] == -7).all()) and bool((k_all[pad + n:] == -7).all())
    assert bool((r_all[:pad] == 0xCD).all()) and bool((r_all[pad + n:] == 0xCD).all())
    assert bool((ws[size:] == fill).all())
    got = r_all[pad:pad + n].cpu()
    src = got[(got != 0xCD).any(dim=1)].contiguous().view(torch.int64)[:, 0]
    assert bool(((src >= 0) & (src < n)).all())
    return src.numel()


@pytest.mark.parametrize("off", [[0, 4_000, 1_000, 5_000], [-5, 1 << 40, 3, 5_000],
                                 [3_000, 2_000, 1_000, 0], [1_500, 1_500, 9_999, 5_000]])
def test_malformed_offsets_stay_inside_the_buffers(off):
    note(f"ranks: offsets {off}")
    _check_inside(off, 5_000, 0, RANK)


@pytest.mark.parametrize("max_keys", [0, BOUND])
@pytest.mark.parametrize("off", [[0, 8_000, 1_000, 9_000], [-5, 1 << 40, 3, 12_000],
                                 [8_000, 4_000, 2_000, 0], [6_000, 6_000, 99_999, 12_000],
                                 [0, 7_000, 0, 7_000]])
def test_malformed_offsets_in_the_partition(off, max_keys):
    """In one launch: with a bound, and without one (a viewer may then hold all records)."""
    note(f"partition: offsets {off}, bound {max_keys}")
    _check_inside(off, 12_000, max_keys, PART)


@pytest.mark.parametrize("n,want,part,per,most", [(8_000, PART, SHORT, 10, 4_096),
                                                  (40_000, SPLIT, 640, 12, 2_048)])
def test_viewers_that_overlap_in_an_overlong_part(n, want, part, per, most):
    """Offsets that give the same records to two viewers, whose first part does not fit in LDS: both
    sort it through the same slices of the workspace, which start out as indexes far below zero. Every
    row written is one of the call's rows, whatever the two leave there."""
    note(f"sort: overlapping overlong parts, {n} records")
    total = n + 5_000
    keys = torch.randint(0, 700, (total,), generator=W.gen("cpu", n, 7))
    at = torch.from_numpy(_sample_positions(n, _parts(0, n, part), per, most))
    keys[at] = torch.randint(1_000, 1_000_000_000, (at.numel(),), generator=W.gen("cpu", n, 8))
    assert int((keys[:n] < 700).sum()) > most
    for fill in (0xEE, 0x7F):
        wrote = _check_inside([0, n, 0, n], total, BOUND if want == PART else n, want, keys, fill)
        assert wrote > most


# ---- calls with viewers of more than 8,192 records, at most 162,560: split by chunks beforehand ----

SPLIT_PART, CHUNK, WHOLE, LONGEST = 640, 3072, 2048, 254 * 640


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("lead", [0, 1, WHOLE, CHUNK - 1])
def test_split_sizes(lead, kind):
    """Viewers around the largest one that is sorted whole, one chunk and several, at offsets that
    put the multiples of a part and a chunk anywhere."""
    sizes = [lead, WHOLE, WHOLE + 1, CHUNK, CHUNK + 1, 0, 20_000, 2 * CHUNK, 1, 16 * SPLIT_PART + 1, 8193]
    _check(sizes, _keys(kind, sum(sizes), lead + 1), f"split, {kind} after {lead}", SPLIT, max_keys=20_000)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [10_241, LONGEST - 1, LONGEST, LONGEST + 1])
def test_split_range_of_lengths(n, kind):
    """Around the shortest single viewer that takes two launches and the longest whose parts are of 640
    records, and the bound from which they are taken."""
    _check([777, n, 5_000], _keys(kind, n + 5_777, 3), f"{kind}, longest {n}", SPLIT, max_keys=n)
    _check([n], _keys(kind, n, 4), f"{kind}, one viewer of {n}", SPLIT)
    _check([8_193, 5_000], _keys(kind, 13_193, 5), f"{kind}, bound 8,193", SPLIT, max_keys=8_193)
    _check([8_192, 5_000], _keys(kind, 13_192, 5), f"{kind}, bound 8,192", PART, max_keys=8_192)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("lead,n", [(0, 1 << 19), (777, 128 * CHUNK), (777, 128 * CHUNK + 1), (3_071, 165_000),
                                    (500, 263_000)])
def test_long_viewers_without_a_bound(lead, n, kind):
    """Viewers of 256 parts that are longer than 640 records, some of them overlong, up to 172 chunks,
    among short ones; the longest call that may take two launches without a bound, and one record more."""
    sizes = [lead] + [n] + [70] * min(100, ((1 << 19) - lead - n) // 70)
    _check(sizes, _keys(kind, sum(sizes), n), f"{n} {kind} after {lead}", SPLIT)
    if n == 1 << 19:
        _check([n, 1], _keys(kind, n + 1, n), f"{n} and 1 {kind}", MERGE)


@pytest.mark.parametrize("kind", ["ids", "wide"])
def test_several_long_viewers_without_a_bound(kind):
    """Each cut into 256 parts of its own length; and ordinary lists of a call of that size."""
    _check([170_000, 0, 180_001, 5, 163_841], _keys(kind, 513_847, 2), f"three long, {kind}", SPLIT)
    _check([5_000] * 64, _keys(kind, 320_000, 2), f"64 x 5,000, {kind}", SPLIT)


@pytest.mark.parametrize("dup", [1, 300, 3_000])
def test_split_keys_that_crowd(dup):
    """Most keys in a sliver of the span (the histogram of the sample can't tell them apart), a few
    far away, some repeated `dup` times."""
    n = 60_000
    keys = torch.arange(n) // dup
    keys[::1000] = (1 << 62) - torch.arange(60)
    keys[7::1000] = -(1 << 62) + torch.arange(60)
    keys = keys[torch.randperm(n, generator=W.gen("cpu", dup, 1))]
    _check([n, 9_000], torch.cat([keys, _keys("ids", 9_000, 2)]), f"crowded, {dup}", SPLIT, max_keys=n)


@pytest.mark.parametrize("lead", [0, 777])
@pytest.mark.parametrize("n", [33_333, 150_000, 300_000])
def test_split_part_that_the_sample_misjudged(n, lead):
    keys = _misjudged(n, min(_parts(lead, n, SPLIT_PART), 256), 12, WHOLE)
    _check([lead, n], torch.cat([_keys("ids", lead, 1), keys]), f"split, misjudged after {lead}", SPLIT,
           max_keys=n)


@pytest.mark.parametrize("row", [16, 144])
@pytest.mark.parametrize("kind", ["spread", "repeats", "two", "equal"])
@pytest.mark.parametrize("extra", [1_800, 2_200, 5_000, 7_300, 9_000])
def test_split_overlong_part_in_pieces(extra, kind, row):
    """One part of a little more than LDS holds up to more than four times that, its records spread,
    repeated, in two far groups, or all alike (a share of its key span that does not fit either)."""
    n = 60_000
    g = W.gen("cpu", extra, 7)
    keys = torch.randint(0, 1 << 40, (n,), generator=g)
    free = torch.ones(n, dtype=torch.bool)
    free[torch.from_numpy(_sample_positions(n, _parts(0, n, SPLIT_PART), 12, WHOLE))] = False
    at = free.nonzero()[:, 0]
    at = at[torch.randperm(at.numel(), generator=g)[:extra]]
    wide = (1 << 40) // 2_000                    # a fifth of a part's share of the span
    v = {"spread": torch.randint(0, wide, (extra,), generator=g),
         "repeats": torch.randint(0, 40, (extra,), generator=g) * (wide // 40),
         "two": torch.randint(0, 2, (extra,), generator=g) * wide,
         "equal": torch.zeros(extra, dtype=torch.int64)}[kind]
    keys[at] = (1 << 39) + v
    inside = int(((keys >= 1 << 39) & (keys <= (1 << 39) + wide)).sum())
    assert inside >= extra
    _check([n, 300], torch.cat([keys, _keys("ids", 300, 1)]), f"part of {inside} {kind}", SPLIT, row=row,
           max_keys=n)


def test_split_viewers_above_the_bound_are_copied_through():
    sizes = [30_000, 9_000, 300, 50_000, 8_200]
    ko = torch.tensor([0] + np.cumsum(sizes).tolist(), dtype=torch.int64)
    n = int(ko[-1])
    keys = _keys("few", n, 1)
    rows = torch.arange(n, dtype=torch.int64).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    note("split sort: bound 9,000")
    assert choice(sizes, 9_000) == SPLIT
    gk, gr = _sort(ko, keys, rows, 9_000)
    wk, wr = oracle.sort_affinity(ko, keys, rows)
    for v, size in enumerate(sizes):
        sl = slice(int(ko[v]), int(ko[v + 1]))
        want = (keys.numpy()[sl], rows.numpy()[sl]) if size > 9_000 else (wk[sl], wr[sl])
        assert np.array_equal(gk[sl], want[0]) and np.array_equal(gr[sl], want[1]), f"viewer {v}"


@pytest.mark.parametrize("off", [[0, 40_000, 10_000, 50_000], [-5, 1 << 40, 3, 50_000],
                                 [30_000, 20_000, 10_000, 0], [0, 20_000, 7, 30_000]])
def test_split_malformed_offsets_stay_inside_the_buffers(off):
    """Viewers that overlap write each other's chunk tables; whatever they hold, what is read and
    written stays inside the call's buffers."""
    note(f"split sort: offsets {off}")
    _check_inside(off, 50_000, 50_000, SPLIT)


@pytest.mark.parametrize("off", [[0, 400_000, 100_000, 500_000], [-5, 1 << 40, 3, 500_000],
                                 [300_000, 200_000, 100_000, 0], [0, 400_000, 0, 400_000]])
def test_split_malformed_offsets_of_long_viewers(off):
    """The same with viewers of 256 longer parts, some of them overlong."""
    note(f"split sort: offsets {off}")
    _check_inside(off, 500_000, 0, SPLIT)
