"""GPU parity of the join's partial sub-tiles, run-time row widths and pad slots against the oracle:
sizes around a sub-tile of 256 candidates and a wavefront, output strides, and the bytes that a
partial sub-tile must leave alone."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2609_22441_amd as P
import workload as W
from gpu_common import FILL, note
from kernel_choice import plain_copy, least_fences

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
WIDTHS = [(64, 32), (128, 64), (128, 128), (48, 80), (16, 16), (208, 96), (1040, 32), (32, 1040)]
GUARD = 300              # rows behind the output


def _case(sizes, wd, we, L, seed, n_docs=500):
    g = W.gen("cpu", seed, 4)
    author = torch.randint(0, 60, (n_docs,), generator=g)
    doc = torch.randint(0, 256, (n_docs, wd), generator=g, dtype=torch.int64).to(torch.uint8)
    reqs = []
    for n in sizes:
        keys = torch.sort(torch.randperm(60, generator=g)[:25]).values
        edge = torch.randint(0, 256, (25, we), generator=g, dtype=torch.int64).to(torch.uint8)
        cand = torch.randint(0, n_docs, (n,), generator=g)
        cand[torch.rand(n, generator=g) < 0.1] = -1
        actor = torch.randint(-1, 60, (n,), generator=g) if L == 2 else None
        reqs.append(W.Request(keys, edge, cand, actor))
    default = torch.randint(0, 256, (we,), generator=g, dtype=torch.int64).to(torch.uint8)
    return author, doc, W.pack(reqs), default


def _check(sizes, wd, we, L, seed, stride, use_default, what):
    note(f"join tails: {what}")
    author, doc, b, default = _case(sizes, wd, we, L, seed)
    store = P.cc_store_create(author.to(DEV), doc.to(DEV))
    try:
        d = b.to(DEV)
        total = b.cand_idx.numel()
        out = torch.full((total + GUARD, stride), FILL, dtype=torch.uint8, device=DEV)
        hit = torch.full((total + GUARD, L), -7, dtype=torch.int8, device=DEV)
        df = default.to(DEV) if use_default else None
        if len(sizes) == 1 and L == 1:
            P.cc_join(store, d.cand_idx, d.keys, d.edge_rows, out, hit, default_row=df)
        else:
            P.cc_join_batched(store, d.cand_offsets, d.cand_idx, d.key_offsets, d.keys, d.edge_rows,
                              out, hit, default_row=df, extra_keys=[d.actor] if L == 2 else None)
        torch.cuda.synchronize()
        wo, wh, inv = oracle.join(author, doc, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys,
                                  b.edge_rows, default_row=default if use_default else None,
                                  n_lookups=L, extra_keys=[b.actor] if L == 2 else None,
                                  out_stride=stride, fill=FILL)
        go, gh = out.cpu().numpy(), hit.cpu().numpy()
        assert np.array_equal(go[:total], wo), f"{what}: rows"
        assert np.array_equal(gh[:total], wh), f"{what}: hits"
        assert (go[total:] == FILL).all() and (gh[total:] == -7).all(), f"{what}: past the end"
        assert P.cc_store_invalid_count(store) == inv, f"{what}: invalid count"
    finally:
        P.cc_store_destroy(store)


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("wd,we", WIDTHS)
def test_one_viewer_sizes_around_a_sub_tile(wd, we, L):
    for n in (1, 63, 65, 255, 256, 257, 513, 1031):
        _check([n], wd, we, L, n, wd + L * we, n % 2 == 0, f"{n} candidates, {wd}+{we} x{L}")


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("wd,we", WIDTHS)
def test_ragged_viewers_with_a_stride(wd, we, L):
    """Segments of 0 to 700 candidates and rows inside a wider stride."""
    sizes = [0, 1, 700, 256, 3, 0, 257, 64, 511, 2, 90]
    _check(sizes, wd, we, L, 9, wd + L * we + 48, True, f"ragged, {wd}+{we} x{L}, stride +48")


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("n", [60_000, 90_000])
def test_short_rows_with_gaps_by_either_copy(n, L):
    """Short rows with gaps, below and above the size of the output up to which they are copied without
    the pipeline; one viewer's candidates end inside a sub-tile."""
    assert plain_copy(n, 96, 16 + 16 * L) == (n == 60_000)
    _check([n - 9_001, 9_001], 16, 16, L, 3, 96, L == 2, f"{n} rows at 96, x{L}")


def test_stride_past_a_sub_tiles_offsets():
    """Strides too long for 32-bit offsets within a sub-tile take the plain copy."""
    for wd, we in ((128, 64), (48, 80)):
        _check([3], wd, we, 1, 2, (1 << 22) + 16, False, f"4 MiB stride, {wd}+{we}")
        _check([3], wd, we, 1, 2, 1 << 22, False, f"4 MiB stride less 16, {wd}+{we}")


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("wd,we", [(128, 64), (48, 80), (1040, 32)])
@pytest.mark.parametrize("n_max", [1, 64, 130, 700])
def test_pad_slots(n_max, wd, we, L):
    """Viewers below, at and above n_max, empty ones; no candidates at all; rows in a stride."""
    for sizes in ([0, 1, 700, 64, 130, 0, 129, 63], [0, 0, 0], [40] * 1_100):
        if n_max == 700 and len(sizes) > 1_000:
            continue
        what = f"{len(sizes)} viewers, n_max {n_max}, {wd}+{we} x{L}"
        note(f"pad slots: {what}")
        author, doc, b, _ = _case(sizes, wd, we, L, n_max)
        store = P.cc_store_create(author.to(DEV), doc.to(DEV))
        try:
            d, B, stride = b.to(DEV), len(sizes), wd + L * we + 16
            out = torch.full((B * n_max + GUARD, stride), FILL, dtype=torch.uint8, device=DEV)
            hit = torch.full((B * n_max + GUARD, L), -7, dtype=torch.int8, device=DEV)
            valid = torch.full((B * n_max + GUARD,), -7, dtype=torch.int8, device=DEV)
            P.cc_join_batched_padded(store, d.cand_offsets, d.cand_idx, d.key_offsets, d.keys,
                                     d.edge_rows, n_max, out, hit, valid,
                                     extra_keys=[d.actor] if L == 2 else None)
            torch.cuda.synchronize()
            wo, wh, _ = oracle.join(author, doc, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys,
                                    b.edge_rows, n_lookups=L,
                                    extra_keys=[b.actor] if L == 2 else None)
            want = np.zeros((B * n_max + GUARD, wd + L * we), np.uint8)
            want_hit = np.zeros((B * n_max + GUARD, L), np.int8)
            want_valid = np.zeros(B * n_max + GUARD, np.int8)
            want[B * n_max:], want_hit[B * n_max:], want_valid[B * n_max:] = FILL, -7, -7
            off = b.cand_offsets.numpy()
            for v, n in enumerate(sizes):
                m = min(n, n_max)
                want[v * n_max:v * n_max + m] = wo[off[v]:off[v] + m]
                want_hit[v * n_max:v * n_max + m] = wh[off[v]:off[v] + m]
                want_valid[v * n_max:v * n_max + m] = 1
            go = out.cpu().numpy()
            assert np.array_equal(go[:, :wd + L * we], want), f"{what}: rows"
            assert (go[:, wd + L * we:] == FILL).all(), f"{what}: stride padding"
            assert np.array_equal(hit.cpu().numpy(), want_hit), f"{what}: hits"
            assert np.array_equal(valid.cpu().numpy(), want_valid), f"{what}: valid"
        finally:
            P.cc_store_destroy(store)


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("wd,we", [(128, 64), (48, 80)])
@pytest.mark.parametrize("viewers", [2, 3, 7, 12, 100, 255, 256, 257])
def test_ranges_by_viewers(viewers, wd, we, L):
    """Small launches whose ranges are a multiple of the viewers (idle workgroups behind them, ranges of
    one candidate) and, past 256 viewers, are not; equal viewers and ragged ones."""
    for sizes in ([1] * viewers, [160] * viewers, [(37 * v + 11) % 301 for v in range(viewers)],
                  [0] * (viewers - 1) + [700]):
        _check(sizes, wd, we, L, viewers, wd + L * we, True, f"{viewers} viewers of {sizes[:3]}.., x{L}")


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("viewers", [78, 79])
def test_few_candidates_of_many_long_lists(viewers, L):
    """Either side of the line past which short segments stage few fences: windows of 16 keys below
    it, and searches between fences 128 keys apart above."""
    k, n_docs = 40_000, 3_000
    assert least_fences(viewers, k) == (4_096 if viewers == 78 else 512)
    note(f"join: {viewers} viewers of {k} keys, {L} lookups")
    g = W.gen("cpu", viewers, 4)
    author = torch.randint(-5, 2 * k + 5, (n_docs,), generator=g)
    doc = torch.randint(0, 256, (n_docs, 48), generator=g, dtype=torch.int64).to(torch.uint8)
    sizes = [(7 * v) % 41 for v in range(viewers)]
    reqs = []
    for n in sizes:
        keys = 2 * torch.arange(k) + torch.randint(0, 2, (k,), generator=g)
        edge = torch.arange(k).repeat_interleave(2).view(torch.uint8).reshape(k, 16)
        cand = torch.randint(-1, n_docs, (n,), generator=g)
        actor = torch.randint(-1, 2 * k, (n,), generator=g) if L == 2 else None
        reqs.append(W.Request(keys, edge, cand, actor))
    b = W.pack(reqs)
    store = P.cc_store_create(author.to(DEV), doc.to(DEV))
    try:
        d, total = b.to(DEV), sum(sizes)
        out = torch.full((total + GUARD, 48 + 16 * L), FILL, dtype=torch.uint8, device=DEV)
        hit = torch.full((total + GUARD, L), -7, dtype=torch.int8, device=DEV)
        P.cc_join_batched(store, d.cand_offsets, d.cand_idx, d.key_offsets, d.keys, d.edge_rows, out,
                          hit, extra_keys=[d.actor] if L == 2 else None)
        torch.cuda.synchronize()
        wo, wh, _ = oracle.join(author, doc, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys,
                                b.edge_rows, n_lookups=L, extra_keys=[b.actor] if L == 2 else None)
        assert np.array_equal(out.cpu().numpy()[:total], wo)
        assert np.array_equal(hit.cpu().numpy()[:total], wh) and 0.3 < wh.mean() < 0.7
        assert bool((out[total:] == FILL).all()) and bool((hit[total:] == -7).all())
    finally:
        P.cc_store_destroy(store)
