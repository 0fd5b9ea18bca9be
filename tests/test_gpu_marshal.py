"""The binding's native marshalling (csrc/marshal.c) against binding.py's own checks: plain calls
give the same results by either, and what is not a plain call is answered the same with the
native path in front as without it."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2609_22441_amd as P
import workload as W
from gpu_common import note

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


class _Off:
    """A marshal module that answers None to everything."""
    def __getattr__(self, name):
        return lambda *a: None


@pytest.fixture(params=["native", "checks"])
def path(request, monkeypatch):
    if request.param == "checks":
        monkeypatch.setattr(P.lib(), "marshal", _Off())
    return request.param


@pytest.fixture
def case():
    s, r = W.shape(4, store_n_docs=2_000, store_n_authors=9_000, req_k=70, req_n_cand=500,
                   req_n_viewers=3)
    st = W.make_store(s, 1, device="cpu")
    b = W.pack(W.make_requests(st, r, 1)).to(DEV)
    store = P.cc_store_create(st.author_id.to(DEV), st.doc_rows.to(DEV))
    yield st, b, store
    P.cc_store_destroy(store)


def _outputs(n, w, L):
    return (torch.full((n, w), 0xCD, dtype=torch.uint8, device=DEV),
            torch.full((n, L), -7, dtype=torch.int8, device=DEV))


def test_plain_calls(path, case):
    """Every entry point with a native path, on torch's current stream, a stream object and a
    handle; results are compared with each other and the store's rows."""
    note(f"marshal: plain calls, {path}")
    st, b, store = case
    side = torch.cuda.Stream()
    results = []
    for stream in (None, side, side.cuda_stream):
        torch.cuda.synchronize()
        n = b.cand_idx.numel()
        o1, h1 = _outputs(n, 192, 1)
        o2, h2 = _outputs(n, 256, 2)
        o3, h3 = _outputs(n, 192, 1)
        o4, h4 = _outputs(3 * 510, 256, 2)
        v4 = torch.full((3 * 510,), -7, dtype=torch.int8, device=DEV)
        ids = st.author_id.to(DEV)[b.cand_idx]
        k0 = int(b.key_offsets[1])
        torch.cuda.synchronize()
        P.cc_join(store, b.cand_idx, b.keys[:k0], b.edge_rows[:k0], o1, h1, stream=stream)
        P.cc_join_batched(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys, b.edge_rows, o2,
                          h2, extra_keys=[b.actor], stream=stream)
        P.cc_join_batched(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys, b.edge_rows, o3,
                          h3, default_row=b.edge_rows[0], author_ids=ids, stream=stream)
        P.cc_join_batched_padded(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys,
                                 b.edge_rows, 510, o4, h4, v4, extra_keys=[b.actor], stream=stream)
        torch.cuda.synchronize()
        results.append([t.cpu() for t in (o1, h1, o2, h2, o3, h3, o4, h4, v4)])
    for r in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(results[0], r))
    out = results[0][2]
    assert torch.equal(out[:, :128], st.doc_rows[b.cand_idx.cpu()].view(torch.uint8))
    assert torch.equal(results[0][6].reshape(3, 510, 256)[:, :500].reshape(-1, 256), out)
    assert torch.equal(results[0][4][:, :128], out[:, :128])


def test_index_and_sort(path):
    note(f"marshal: index and sort, {path}")
    idx = P.cc_store_create_indexed(100, 32)
    try:
        ids = torch.arange(50, device=DEV) * 3
        rows = torch.randint(0, 256, (50, 32), device=DEV).to(torch.uint8)
        ws = torch.empty(P.cc_upsert_workspace_bytes(50), dtype=torch.uint8, device=DEV)
        assert P.cc_store_upsert(idx, ids, ids, rows, ws) == (50, 0)
        assert P.cc_store_upsert(idx, ids, ids, rows, ws) == (0, 0)
        pos = torch.empty(51, dtype=torch.int64, device=DEV)
        P.cc_resolve_ids(idx, torch.cat([ids, ids[:1] + 1]), pos)
        assert pos.tolist() == list(range(50)) + [-1]
        with pytest.raises(P.CCError) as e:
            P.cc_store_upsert(idx, ids + 10_000, ids, rows, ws[:8])
        assert e.value.status == 1
        with pytest.raises(ValueError):
            P.cc_store_upsert(idx, ids, ids[:49], rows, ws)
        with pytest.raises(ValueError):
            P.cc_store_upsert(idx, ids, ids, rows[:, :16].contiguous(), ws)
        with pytest.raises(ValueError):
            P.cc_resolve_ids(idx, ids, pos[:10])
    finally:
        P.cc_store_destroy(idx)
    off = torch.tensor([0, 30, 50], device=DEV)
    keys = torch.randint(0, 40, (50,), device=DEV)
    k, r = torch.empty_like(keys), torch.empty_like(rows)
    ws = torch.empty(P.cc_sort_workspace_bytes(50, 2), dtype=torch.uint8, device=DEV)
    for kw in ({}, {"max_keys": 30}, {"method": P.SORT_RADIX, "key_bits": 9}):
        k.fill_(-1)
        P.cc_sort_affinity(off, keys, rows, k, r, ws, **kw)
        for a, b in ((0, 30), (30, 50)):
            order = np.argsort(keys[a:b].cpu().numpy(), kind="stable")
            assert torch.equal(k[a:b].cpu(), keys[a:b].cpu()[order])
            assert torch.equal(r[a:b].cpu(), rows[a:b].cpu()[order])
    with pytest.raises(P.CCError):
        P.cc_sort_affinity(off, keys, rows, k, r, ws[:16])
    with pytest.raises(ValueError):
        P.cc_sort_affinity(off, keys, rows, k[:40], r, ws)
    with pytest.raises(P.CCError):
        P.cc_sort_affinity(off, keys, rows, k, r, ws, key_bits=65)


def test_what_is_not_plain(path, case):
    """Wrong types, layouts, sizes and devices raise as ever; 3-D rows, raw pointers, tensor
    subclasses and explicit totals still work."""
    note(f"marshal: not plain, {path}")
    st, b, store = case
    n = b.cand_idx.numel()
    k0 = int(b.key_offsets[1])
    keys, edge = b.keys[:k0], b.edge_rows[:k0]

    def join(cand=b.cand_idx, keys=keys, edge=edge, out=None, hit=None, **kw):
        o, h = _outputs(n, 192, 1)
        P.cc_join(store, cand, keys, edge, o if out is None else out, h if hit is None else hit, **kw)
        torch.cuda.synchronize()
        return o.cpu(), h.cpu()

    want = join()
    for bad, exc in ((dict(cand=b.cand_idx.int()), TypeError), (dict(cand=b.cand_idx.cpu()), ValueError),
                     (dict(keys=keys.cpu()), ValueError), (dict(edge=edge[:-1]), ValueError),
                     (dict(cand=b.cand_idx.repeat(2)[::2]), ValueError),
                     (dict(out=torch.empty(n, 176, dtype=torch.uint8, device=DEV)), ValueError),
                     (dict(out=torch.empty(n - 1, 192, dtype=torch.uint8, device=DEV)), ValueError),
                     (dict(out=torch.empty(192, n, dtype=torch.uint8, device=DEV).t()), ValueError),
                     (dict(out=torch.empty(n, 200, dtype=torch.uint8, device=DEV)[:, 4:196]), P.CCError),
                     (dict(hit=torch.empty(n, dtype=torch.uint8, device=DEV)), TypeError),
                     (dict(default_row=edge[0][:8]), ValueError)):
        with pytest.raises(exc):
            join(**bad)
    assert all(torch.equal(x, y) for x, y in zip(join(edge=edge.reshape(k0, 8, 4)), want))

    class Sub(torch.Tensor):
        pass

    assert all(torch.equal(x, y) for x, y in zip(join(cand=b.cand_idx.as_subclass(Sub)), want))
    o, h = _outputs(n, 256, 2)
    P.cc_join_batched(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys, b.edge_rows, o, h,
                      extra_keys=[b.actor], total_cand=n, total_keys=b.keys.numel())
    o3 = torch.empty(3, 500, 256, dtype=torch.uint8, device=DEV)
    h3 = torch.empty(3, 500, 2, dtype=torch.int8, device=DEV)
    v3 = torch.empty(3, 500, dtype=torch.int8, device=DEV)
    P.cc_join_batched_padded(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys, b.edge_rows,
                             500, o3, h3, v3, extra_keys=[b.actor])
    torch.cuda.synchronize()
    assert torch.equal(o3.reshape(n, 256).cpu(), o.cpu())
    with pytest.raises(ValueError):
        P.cc_join_batched(store, b.cand_offsets, b.cand_idx, b.key_offsets[:2], b.keys, b.edge_rows,
                          o, h, extra_keys=[b.actor])
    with pytest.raises(ValueError):
        P.cc_join_batched(store, b.cand_offsets, b.cand_idx, b.key_offsets, b.keys, b.edge_rows,
                          o, h, extra_keys=[b.actor[:-1]])
