"""GPU parity of the partition sort (cc_sort_affinity's choice for viewers of moderate length)
against the oracle's stable sort: sizes around a part, the LDS tile and the sample; key
distributions that break the sample's estimate; bounds; malformed offsets; and the same of the split
method that calls with long viewers take."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2609_22441_amd as P
import workload as W
from gpu_common import note

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

PART = 1024              # records per part in calls of at most 2^18 records


def _sort(ko, keys, rows, max_keys=0):
    n = keys.numel()
    ws = torch.full((max(16, P.cc_sort_workspace_bytes(n, ko.numel() - 1)),), 0xEE,
                    dtype=torch.uint8, device=DEV)
    k_out = torch.full((n,), -7, dtype=torch.int64, device=DEV)
    r_out = torch.full(rows.shape, 0xCD, dtype=torch.uint8, device=DEV)
    P.cc_sort_affinity(ko.to(DEV), keys.to(DEV), rows.to(DEV), k_out, r_out, ws, max_keys=max_keys)
    torch.cuda.synchronize()
    return k_out.cpu().numpy(), r_out.cpu().numpy()


def _check(sizes, keys, what, row=16, max_keys=0):
    note(f"partition sort: {what}")
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
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["ids", "few", "equal", "ascending", "descending", "wide"])
@pytest.mark.parametrize("n", [1, 65, 513, PART, PART + 1, 4097, 9_001, 20_011, 140_003])
def test_one_viewer(n, kind):
    _check([n], _keys(kind, n, n), f"one viewer, {n} {kind} records", row=48 if n < 5000 else 16)


@pytest.mark.parametrize("kind", ["ids", "few", "equal", "ascending", "descending", "wide"])
@pytest.mark.parametrize("n", [1, 513, PART, PART + 1, 4097])
def test_one_viewer_beside_a_long_one(n, kind):
    """The same with a 40,000-record viewer in the call: above the size whose ranks are counted by
    comparison, so that both viewers are cut into parts."""
    _check([n, 40_000], _keys(kind, n + 40_000, n), f"{n} and 40,000 {kind} records")


@pytest.mark.parametrize("bits", [31, 40, 52, 53, 63])
def test_ranks_with_and_without_room_for_the_position(bits):
    """Keys whose span leaves just enough, and just too few, bits for a record's position in one
    word (n = 1,500: 11 bits), in two groups that lanes alternate between."""
    g = W.gen("cpu", bits, 3)
    keys = torch.randint(0, 40, (1_500,), generator=g)
    keys[1::2] += 1 << (bits - 1)
    _check([1_500, 130], torch.cat([keys, _keys("few", 130, 1)]), f"two groups, bit {bits - 1}")


@pytest.mark.parametrize("row", [16, 32, 80, 128, 16 * 513])
def test_row_widths(row):
    n = 2_500 if row < 1000 else 700
    _check([n, 0, 300], _keys("ids", n + 300, row), f"row width {row}", row=row)


@pytest.mark.parametrize("max_keys", [0, 30_000])
def test_ragged_viewers(max_keys):
    """Viewers that start and end anywhere against the multiples of a part, empty ones included;
    the call is above 2^18 records, so the longer parts are used."""
    g = W.gen("cpu", 8, 3)
    sizes = torch.cat([torch.tensor([0, 1, 1023, 1024, 1025, 1536, 1537, 30_000, 0, 4096, 4097]),
                       torch.randint(0, 9_000, (80,), generator=g), torch.tensor([0, 2, 0])])
    n = int(sizes.sum())
    assert n > 1 << 18
    _check(sizes, _keys("ids", n, 9), f"ragged, max_keys {max_keys}", max_keys=max_keys)


def test_more_viewers_than_one_search_round():
    g = W.gen("cpu", 9, 3)
    sizes = torch.randint(0, 12, (1_700,), generator=g)
    sizes[::230] = 3_000
    _check(sizes, _keys("few", int(sizes.sum()), 3), "1,700 viewers")


def test_above_the_radix_threshold_with_a_bound():
    """2^20 records and more in viewers that the caller bounds by 2^17 or less."""
    _check([60_000] * 18, _keys("ids", 18 * 60_000, 4), "18 x 60,000", max_keys=60_000)


def _sample_positions(n, parts, per=10, most=4096):
    """The kernel's sample: one hashed position per stratum."""
    s = min(most if parts > most // per else max(64, parts * per), n)
    i = np.arange(s, dtype=np.uint64)
    step = np.uint64((n << 12) // s)
    a, b = (i * step) >> np.uint64(12), ((i + np.uint64(1)) * step) >> np.uint64(12)
    h = (i * np.uint64(2654435761)) & np.uint64(0xFFFFFFFF)
    return (a + ((h * (b - a)) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("lead", [0, 777])
@pytest.mark.parametrize("n", [20_000, 33_333])
def test_part_that_the_sample_misjudged(n, lead):
    """Every sampled record outside the band that all others share: one part then holds far more
    records than LDS does and is sorted through the workspace."""
    parts = 1 + (lead + n - 1) // PART - lead // PART
    g = W.gen("cpu", n, 7)
    keys = 500_000_000 + torch.randint(0, 700, (n,), generator=g)        # repeats in the band
    at = torch.from_numpy(_sample_positions(n, parts))
    keys[at] = torch.randint(0, 1_000_000_000, (at.numel(),), generator=g)
    band = (keys >= 500_000_000) & (keys < 500_000_700)
    assert int(band.sum()) > 2 * 4096 - 1000
    _check([lead, n], torch.cat([_keys("ids", lead, 1), keys]), f"misjudged part, {n} after {lead}")


@pytest.mark.parametrize("max_keys", [1, 1024, 6000])
def test_viewers_above_the_bound_are_copied_through(max_keys):
    sizes = [5000, 20_000, 300, 0, 6001, 1]
    ko = torch.tensor([0] + np.cumsum(sizes).tolist(), dtype=torch.int64)
    n = int(ko[-1])
    keys = _keys("few", n, max_keys)
    rows = torch.arange(n, dtype=torch.int64).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    note(f"partition sort: bound {max_keys}")
    gk, gr = _sort(ko, keys, rows, max_keys)
    wk, wr = oracle.sort_affinity(ko, keys, rows)
    for v, size in enumerate(sizes):
        sl = slice(int(ko[v]), int(ko[v + 1]))
        want = (keys.numpy()[sl], rows.numpy()[sl]) if size > max_keys else (wk[sl], wr[sl])
        assert np.array_equal(gk[sl], want[0]), f"viewer {v} ({size}): keys"
        assert np.array_equal(gr[sl], want[1]), f"viewer {v} ({size}): rows"


def test_malformed_offsets_stay_inside_the_buffers():
    """Offsets out of order and out of range: the output is unspecified, but the bytes around it
    stay as they were and every row written is one of the call's rows."""
    note("partition sort: malformed offsets")
    n, pad = 5_000, 4_096
    for off in ([0, 4_000, 1_000, n], [-5, 1 << 40, 3, n], [3_000, 2_000, 1_000, 0],
                [1_500, 1_500, 9_999, n]):
        ko = torch.tensor(off, dtype=torch.int64)
        keys = _keys("ids", n, 2)
        rows = torch.arange(n).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
        k_all = torch.full((n + 2 * pad,), -7, dtype=torch.int64, device=DEV)
        r_all = torch.full((n + 2 * pad, 16), 0xCD, dtype=torch.uint8, device=DEV)
        ws = torch.zeros(P.cc_sort_workspace_bytes(n, 3), dtype=torch.uint8, device=DEV)
        P.cc_sort_affinity(ko.to(DEV), keys.to(DEV), rows.to(DEV), k_all[pad:pad + n],
                           r_all[pad:pad + n], ws)
        torch.cuda.synchronize()
        assert bool((k_all[:pad] == -7).all()) and bool((k_all[pad + n:] == -7).all())
        assert bool((r_all[:pad] == 0xCD).all()) and bool((r_all[pad + n:] == 0xCD).all())
        got = r_all[pad:pad + n].cpu()
        wrote = (got != 0xCD).any(dim=1)
        src = got[wrote].contiguous().view(torch.int64)[:, 0]
        assert bool(((src >= 0) & (src < n)).all())


# ---- calls with viewers of more than 8,192 records, at most 162,560: split by chunks beforehand ----

SPLIT, CHUNK, WHOLE, LONGEST = 640, 3072, 2048, 254 * 640


@pytest.mark.parametrize("kind", ["ids", "few", "equal", "ascending", "descending", "wide"])
@pytest.mark.parametrize("lead", [0, 1, WHOLE, CHUNK - 1])
def test_split_sizes(lead, kind):
    """Viewers around the largest one that is sorted whole, one chunk and several, at offsets that
    put the multiples of a part and a chunk anywhere."""
    sizes = [lead, WHOLE, WHOLE + 1, CHUNK, CHUNK + 1, 0, 20_000, 2 * CHUNK, 1, 16 * SPLIT + 1, 8193]
    _check(sizes, _keys(kind, sum(sizes), lead + 1), f"split, {kind} after {lead}", max_keys=20_000)


@pytest.mark.parametrize("kind", ["ids", "few", "wide"])
@pytest.mark.parametrize("n", [8_193, LONGEST, LONGEST + 1])
def test_split_range_of_lengths(n, kind):
    _check([777, n, 5_000], _keys(kind, n + 5_777, 3), f"{kind}, longest {n}", max_keys=n)
    _check([n], _keys(kind, n, 4), f"{kind}, one viewer of {n}")


@pytest.mark.parametrize("dup", [1, 300, 3_000])
def test_split_keys_that_crowd(dup):
    """Most keys in a sliver of the span (the histogram of the sample can't tell them apart), a few
    far away, some repeated `dup` times."""
    n = 60_000
    keys = torch.arange(n) // dup
    keys[::1000] = (1 << 62) - torch.arange(60)
    keys[7::1000] = -(1 << 62) + torch.arange(60)
    keys = keys[torch.randperm(n, generator=W.gen("cpu", dup, 1))]
    _check([n, 9_000], torch.cat([keys, _keys("ids", 9_000, 2)]), f"crowded, {dup}", max_keys=n)


@pytest.mark.parametrize("lead", [0, 777])
def test_split_part_that_the_sample_misjudged(lead):
    n = 33_333
    parts = 1 + (lead + n - 1) // SPLIT - lead // SPLIT
    keys = 500_000_000 + torch.randint(0, 700, (n,), generator=W.gen("cpu", n, 7))
    at = torch.from_numpy(_sample_positions(n, parts, 12, WHOLE))
    keys[at] = torch.randint(0, 1_000_000_000, (at.numel(),), generator=W.gen("cpu", n, 8))
    assert int(((keys >= 500_000_000) & (keys < 500_000_700)).sum()) > 2 * WHOLE
    _check([lead, n], torch.cat([_keys("ids", lead, 1), keys]), f"split, misjudged after {lead}",
           max_keys=n)


def test_part_of_a_short_viewer_that_the_sample_misjudged():
    n, lead = 8_000, 6_000                       # viewers of at most 8,192 records: not split
    parts = 1 + (lead + n - 1) // PART - lead // PART
    keys = 500_000_000 + torch.randint(0, 700, (n,), generator=W.gen("cpu", n, 7))
    at = torch.from_numpy(_sample_positions(n, parts))
    keys[at] = torch.randint(0, 1_000_000_000, (at.numel(),), generator=W.gen("cpu", n, 8))
    _check([lead, n], torch.cat([_keys("ids", lead, 1), keys]), "misjudged, 8,000", max_keys=n)


def test_split_viewers_above_the_bound_are_copied_through():
    sizes = [30_000, 9_000, 300, 50_000, 8_200]
    ko = torch.tensor([0] + np.cumsum(sizes).tolist(), dtype=torch.int64)
    n = int(ko[-1])
    keys = _keys("few", n, 1)
    rows = torch.arange(n, dtype=torch.int64).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    note("split sort: bound 9,000")
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
    note("split sort: malformed offsets")
    n, pad = 50_000, 4_096
    keys = _keys("ids", n, 2)
    rows = torch.arange(n).repeat_interleave(2).view(torch.uint8).reshape(n, 16)
    k_all = torch.full((n + 2 * pad,), -7, dtype=torch.int64, device=DEV)
    r_all = torch.full((n + 2 * pad, 16), 0xCD, dtype=torch.uint8, device=DEV)
    size = P.cc_sort_workspace_bytes(n, 3)
    ws = torch.full((size + pad,), 0xEE, dtype=torch.uint8, device=DEV)
    P.cc_sort_affinity(torch.tensor(off).to(DEV), keys.to(DEV), rows.to(DEV), k_all[pad:pad + n],
                       r_all[pad:pad + n], ws[:size], max_keys=50_000)
    torch.cuda.synchronize()
    assert bool((k_all[:pad] == -7).all()) and bool((k_all[pad + n:] == -7).all())
    assert bool((r_all[:pad] == 0xCD).all()) and bool((r_all[pad + n:] == 0xCD).all())
    assert bool((ws[size:] == 0xEE).all())
    got = r_all[pad:pad + n].cpu()
    src = got[(got != 0xCD).any(dim=1)].contiguous().view(torch.int64)[:, 0]
    assert bool(((src >= 0) & (src < n)).all())


@pytest.mark.parametrize("n,part,per,most", [(8_000, PART, 10, 4_096), (40_000, SPLIT, 12, WHOLE)])
def test_viewers_that_overlap_in_an_overlong_part(n, part, per, most):
    """Offsets that give the same records to two viewers, whose first part does not fit in LDS: both
    sort it through the same slices of the workspace, which start out as indexes far below zero. Every
    row written is one of the call's rows, whatever the two leave there."""
    note(f"sort: overlapping overlong parts, {n} records")
    total, pad = n + 5_000, 4_096
    keys = torch.randint(0, 700, (total,), generator=W.gen("cpu", n, 7))
    at = torch.from_numpy(_sample_positions(n, 1 + (n - 1) // part, per, most))
    keys[at] = torch.randint(1_000, 1_000_000_000, (at.numel(),), generator=W.gen("cpu", n, 8))
    assert int((keys[:n] < 700).sum()) > most
    rows = torch.arange(total).repeat_interleave(2).view(torch.uint8).reshape(total, 16)
    k_all = torch.full((total + 2 * pad,), -7, dtype=torch.int64, device=DEV)
    r_all = torch.full((total + 2 * pad, 16), 0xCD, dtype=torch.uint8, device=DEV)
    size = P.cc_sort_workspace_bytes(total, 3)
    for fill in (0xEE, 0x7F):
        ws = torch.full((size + pad,), fill, dtype=torch.uint8, device=DEV)
        P.cc_sort_affinity(torch.tensor([0, n, 0, n]).to(DEV), keys.to(DEV), rows.to(DEV),
                           k_all[pad:pad + total], r_all[pad:pad + total], ws[:size],
                           max_keys=8_192 if part == PART else n)
        torch.cuda.synchronize()
        assert bool((k_all[:pad] == -7).all()) and bool((k_all[pad + total:] == -7).all())
        assert bool((r_all[:pad] == 0xCD).all()) and bool((r_all[pad + total:] == 0xCD).all())
        assert bool((ws[size:] == fill).all())
        got = r_all[pad:pad + total].cpu()
        src = got[(got != 0xCD).any(dim=1)].contiguous().view(torch.int64)[:, 0]
        assert src.numel() > most and bool(((src >= 0) & (src < total)).all())
