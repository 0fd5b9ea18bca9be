"""Timed cases of the edge-feature join library: what a ranking service has it do per request,
per serving batch, per affinity refresh and per ingestion batch, through the public entry points.

Each case is a dict of plain values. ``listed()`` names the fixed ones, ``draw(rng)`` gives more
of the same ranges, ``prepare`` makes what a caller holds before the call (the store, the
request's device buffers, the output buffers), ``run`` is one pass. Every output is a copy of
input bytes or a whole number, so the outputs of two correct implementations are equal.

Five kinds of case:
  join     one cc_join (one viewer) or cc_join_batched launch (several viewers in CSR form)
  padded   cc_join_batched_padded: the same into the padded [B, n_max] layout with a valid mask
  request  document ids resolved to positions (cc_resolve_ids), then joined
  sort     cc_sort_affinity: a viewer's affinity records put in key order with their rows
  ingest   cc_store_upsert, then the new documents read back by id as a request would
"""
from __future__ import annotations

import functools
import math

import torch

import paper_2609_22441_amd as P

DEV = "cuda"
MAX_BYTES = 1_100_000_000       # of the largest listed case: a drawn one stays below


def listed():
    return [
        # A small request: 10,000 candidates from a 1M-document store, 1,000 affinity records,
        # fp32 rows of 16 + 8 columns. Latency and launch cost count.
        _join("join_small", docs=1_000_000, zipf=False, viewers=1, n=10_000, k=1_000, doc=64,
              edge=32, in_net=0.0),
        # One production-shaped request end to end: 50,000 document ids resolved on the index,
        # then joined against 5,000 affinity records (64 + 32 bf16 columns).
        dict(name="request", kind="request", docs=10_000_000, viewers=1, n=50_000, k=5_000,
             doc=128, edge=64, miss=0.02, in_net=0.7),
        # A serving batch of 8 such requests in one launch.
        _join("join_batch_8", viewers=8, n=50_000, k=5_000),
        # The headline step: 64 requests, 3.2M candidates in one launch.
        _join("join_batch_64", viewers=64, n=50_000, k=5_000),
        # Ragged viewers: between 100 and 30,000 affinity records each.
        _join("join_ragged", viewers=64, n=30_000, k_lo=100, k=30_000),
        # A serving batch of uneven requests in the padded layout that a dense model takes;
        # fp32 rows of 12 + 20 columns, a default row for authors without a record.
        dict(name="join_padded", kind="padded", docs=2_000_000, zipf=True, viewers=12, n_lo=9_000,
             n=41_003, k_lo=1_000, k=8_000, doc=48, edge=80, lookups=1, in_net=0.5,
             default_row=True, authors=False, bad=0.01),
        # Second-degree candidates: author and actor looked up in 20,000 records.
        _join("double_join", viewers=1, n=100_000, k=20_000, lookups=2),
        # Very long lists on a store far larger than the caches, every candidate in network.
        _join("join_long_lists", docs=50_000_000, viewers=32, n=31_250, k=100_000, edge=128,
              in_net=1.0),
        # One viewer's affinity records after an update, put in order before the join.
        _sort("sort_request", viewers=1, k=5_000, row=64),
        # A batch of viewers with ragged lists.
        _sort("sort_ragged", viewers=64, k_lo=100, k=30_000, row=64, bound=True),
        # Large lists of many viewers: the bulk refresh (key span known to the caller).
        _sort("sort_large", viewers=32, k=100_000, row=128, ids=50_000_000, bound=True, bits=True),
        # An ingestion batch against an index of 10M documents: 20% new ids on the first pass
        # (every id is stored on a replay), 5% repeats inside the batch.
        dict(name="ingest", kind="ingest", docs=10_000_000, n=300_000, doc=128, new=0.2,
             repeat=0.05),
    ]


def _join(name, docs=10_000_000, zipf=True, viewers=1, n=50_000, n_lo=0, k=5_000, k_lo=0, doc=128,
          edge=64, lookups=1, in_net=0.7, default_row=False, authors=False, bad=0.0):
    return dict(name=name, kind="join", docs=docs, zipf=zipf, viewers=viewers, n_lo=n_lo, n=n,
                k_lo=k_lo, k=k, doc=doc, edge=edge, lookups=lookups, in_net=in_net,
                default_row=default_row, authors=authors, bad=bad)


def _sort(name, viewers=1, k=5_000, k_lo=0, row=64, ids=10_000_000, bound=False, bits=False):
    return dict(name=name, kind="sort", viewers=viewers, k_lo=k_lo, k=k, row=row, ids=ids,
                bound=bound, bits=bits)


# Row widths in bytes: the bf16 and fp32 pairs of the five workload shapes, and others.
WIDTHS = [(64, 32), (128, 64), (128, 128), (128, 64), (48, 16), (16, 48), (48, 80), (192, 96)]


def draw(rng):
    kind = rng.choice(["join", "join", "join", "padded", "request", "sort", "sort", "ingest"])
    while True:
        c = _DRAW[kind](rng)
        c.pop("name", None)
        if work(c)["bytes"] <= MAX_BYTES:
            return c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_join(rng):
    doc, edge = rng.choice(WIDTHS)
    viewers = 1 if rng.random() < 0.3 else _log(rng, 2, 80)
    ragged_n, ragged_k = rng.random() < 0.4, rng.random() < 0.5
    n, k = _log(rng, 5_000, 120_000), _log(rng, 300, 100_000)
    return _join("", docs=_log(rng, 500_000, 20_000_000), zipf=rng.random() < 0.8,
                 viewers=viewers, n=n, n_lo=max(1, n // 8) if ragged_n else 0, k=k,
                 k_lo=max(50, k // 30) if ragged_k and viewers > 1 else 0, doc=doc, edge=edge,
                 lookups=2 if rng.random() < 0.25 else 1, in_net=rng.choice([0.0, 0.5, 0.7, 1.0]),
                 default_row=rng.random() < 0.3, authors=viewers > 1 and rng.random() < 0.25,
                 bad=rng.choice([0.0, 0.02]))


def _draw_padded(rng):
    c = _draw_join(rng)
    return dict(c, kind="padded", viewers=_log(rng, 2, 40), n_lo=max(1, c["n"] // 4),
                authors=False)


def _draw_request(rng):
    doc, edge = rng.choice(WIDTHS)
    return dict(kind="request", docs=_log(rng, 500_000, 10_000_000), viewers=rng.choice([1, 1, 4, 8]),
                n=_log(rng, 5_000, 100_000), k=_log(rng, 300, 20_000), doc=doc, edge=edge,
                miss=rng.choice([0.0, 0.02, 0.1]), in_net=rng.choice([0.0, 0.7]))


def _draw_sort(rng):
    viewers = 1 if rng.random() < 0.3 else _log(rng, 2, 100)
    k = _log(rng, 300, 120_000)
    return _sort("", viewers=viewers, k=k, k_lo=max(50, k // 100) if rng.random() < 0.5 else 0,
                 row=rng.choice([16, 32, 64, 64, 80, 128, 128]),
                 ids=rng.choice([1_000_000, 10_000_000, 50_000_000, 1 << 62]),
                 bound=rng.random() < 0.6, bits=rng.random() < 0.4)


def _draw_ingest(rng):
    return dict(kind="ingest", docs=_log(rng, 500_000, 10_000_000), n=_log(rng, 20_000, 1_000_000),
                doc=rng.choice([64, 128, 48, 192]), new=rng.choice([0.0, 0.2, 1.0]),
                repeat=rng.choice([0.0, 0.05, 0.3]))


_DRAW = {"join": _draw_join, "padded": _draw_padded, "request": _draw_request,
         "sort": _draw_sort, "ingest": _draw_ingest}


# ---- sizes ----------------------------------------------------------------------------------

def _sizes(lo, hi, count, shift):
    """`count` sizes in [lo, hi] (all hi when lo is 0), spread evenly over their logarithm and
    put in a mixed order; the same for every seed, so that a case's work is fixed."""
    if not lo or lo >= hi:
        return [hi] * count
    pos = [((i + shift) * 0.6180339887498949) % 1.0 for i in range(count)]
    return [int(math.exp(math.log(lo) + p * (math.log(hi) - math.log(lo)))) for p in pos]


def _n_k(case):
    b = case["viewers"]
    return (_sizes(case.get("n_lo", 0), case["n"], b, 1), _sizes(case.get("k_lo", 0), case["k"], b, 2))


def work(case):
    """Bytes of one pass with each input read once and each output written once. An edge row is
    counted per distinct row hit, bounded by the lookups that hit and by the rows there are."""
    kind = case["kind"]
    if kind == "sort":
        total = sum(_sizes(case["k_lo"], case["k"], case["viewers"], 2))
        return {"bytes": total * 2 * (8 + case["row"]), "flops": 0}
    if kind == "ingest":
        n, d = case["n"], case["doc"]
        # ids, authors, rows in; row, author and map entry of each record written; then ids to
        # positions and the rows read back.
        return {"bytes": n * (8 + 8 + d + d + 8 + 16) + n * (8 + 16 + 8) + n * (8 + 4 + d + d + 16 + 1),
                "flops": 0}
    ns, ks = _n_k(case)
    lookups = case.get("lookups", 1)
    d, e = case["doc"], case["edge"]
    per = 8 + 4 + d + d + lookups * (e + 1) + (lookups - 1) * 8
    total = sum(n * per + 8 * k for n, k in zip(ns, ks))
    total += sum(min(int(n * case["in_net"]), k) * e for n, k in zip(ns, ks))
    if kind == "request":
        total += sum(ns) * (8 + 16 + 8)
    if kind == "padded":
        total += (len(ns) * max(ns) - sum(ns)) * (d + lookups * e) + len(ns) * max(ns)
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"              # copies of input bytes, and whole numbers


def exact(case, seed):
    return None                 # no output is a computed number


# ---- inputs ---------------------------------------------------------------------------------

class _Store:
    """A store handle that is given back with the state that holds it."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        try:
            torch.cuda.synchronize()
            P.cc_store_destroy(self.handle)
        except Exception:       # the process is ending
            pass


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1_000_003 + stream)
    return g


@functools.lru_cache(maxsize=4)
def _zipf_cdf(m, s):
    """Cumulative weights r^-s of ranks 1..m, summed on the host (in a fixed order)."""
    return torch.cumsum(torch.arange(1, m + 1, dtype=torch.float64).pow_(-s), 0).to(DEV)


def _authors(n, m, zipf, g):
    """Author id per document over [0, m), and the ids in order of popularity (None: uniform)."""
    if not zipf:
        return torch.randint(0, m, (n,), device=DEV, generator=g), None
    cdf = _zipf_cdf(m, 1.1)
    by_rank = torch.randperm(m, device=DEV, generator=g)
    u = torch.rand(n, dtype=torch.float64, device=DEV, generator=g) * cdf[-1]
    return by_rank[torch.searchsorted(cdf, u, right=True).clamp_(max=m - 1)], by_rank


def _rows(n, nbytes, g):
    """n rows of bf16 N(0,1) values as bytes."""
    r = torch.randn(n, nbytes // 2, device=DEV, generator=g, dtype=torch.bfloat16)
    return r.view(torch.uint8)


def _unique(m, count, g):
    """`count` distinct ids of [0, m), in no order."""
    draw = count + count // 8 + 64
    while True:
        x = torch.unique(torch.randint(0, m, (draw,), device=DEV, generator=g))
        if x.numel() >= count:
            return x[torch.randperm(x.numel(), device=DEV, generator=g)[:count]]
        draw *= 2


def _keys(k, m, by_rank, g):
    """k distinct author ids, ascending: half of them among the most popular 1%."""
    if by_rank is None:
        return torch.sort(_unique(m, k, g)).values
    top = max(m // 100, k)
    a = by_rank[_unique(top, k // 2, g)]
    b = _unique(m, k, g)
    b = b[~torch.isin(b, a)]
    return torch.sort(torch.cat([a, b[: k - a.numel()]])).values


def _offsets(sizes):
    off = [0]
    for x in sizes:
        off.append(off[-1] + x)
    return torch.tensor(off, dtype=torch.int64, device=DEV)


def _requests(case, author, by_rank, m, g):
    """Per viewer: keys, candidates (a share in network, the rest over all documents), actors."""
    ns, ks = _n_k(case)
    docs = author.numel()
    order = torch.argsort(author)
    first = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(author, minlength=m), 0, out=first[1:])
    keys, cands, actors = [], [], []
    for n, k in zip(ns, ks):
        key = _keys(k, m, by_rank, g)
        cand = torch.randint(0, docs, (n,), device=DEV, generator=g)
        start, lens = first[key], first[key + 1] - first[key]
        ends = torch.cumsum(lens, 0)
        pool = int(ends[-1])
        n_in = int(n * case["in_net"]) if pool else 0
        if n_in:
            # Pool members evenly spaced from a random start: without repeats when the pool allows.
            step = max(1, pool // n_in)
            u = (torch.arange(n_in, device=DEV) * step
                 + torch.randint(0, pool, (1,), device=DEV, generator=g)) % pool
            j = torch.searchsorted(ends, u, right=True)
            cand[:n_in] = order[start[j] + u - (ends[j] - lens[j])]
        cand = cand[torch.randperm(n, device=DEV, generator=g)]
        if case.get("bad"):
            cand[torch.rand(n, device=DEV, generator=g) < case["bad"]] = -1
        keys.append(key)
        cands.append(cand)
        pick = key[torch.randint(0, k, (n,), device=DEV, generator=g)]
        none = torch.rand(n, device=DEV, generator=g) < 0.5
        actors.append(torch.where(none, torch.full_like(pick, -1), pick))
    return ns, ks, torch.cat(keys), torch.cat(cands), torch.cat(actors)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def _join_state(case, g, author, by_rank, m, handle):
    ns, ks, keys, cand, actor = _requests(case, author, by_rank, m, g)
    lookups = case.get("lookups", 1)
    s = {"kind": case["kind"], "store": handle, "keys": keys, "cand": cand, "edge": _rows(sum(ks), case["edge"], g),
         "cand_offsets": _offsets(ns), "key_offsets": _offsets(ks), "actor": None,
         "authors": None, "default": None}
    if lookups == 2:
        s["actor"] = [actor]
    if case.get("authors"):
        s["authors"] = author[cand.clamp(min=0)]
    if case.get("default_row"):
        s["default"] = _rows(1, case["edge"], g)[0]
    width = case["doc"] + lookups * case["edge"]
    s["n_max"] = max(ns)
    rows = len(ns) * max(ns) if case["kind"] == "padded" else sum(ns)
    s["out"] = torch.empty(rows, width, dtype=torch.uint8, device=DEV)
    s["hit"] = torch.empty(rows, lookups, dtype=torch.int8, device=DEV)
    s["valid"] = torch.empty(rows, dtype=torch.int8, device=DEV)
    return s


def _prepare_join(case, seed):
    g = _gen(seed, 0)
    m = max(1_000, case["docs"] if case["zipf"] else case["docs"] // 10, 4 * case["k"])
    author, by_rank = _authors(case["docs"], m, case["zipf"], g)
    store = _Store(P.cc_store_create(author, _rows(case["docs"], case["doc"], g)))
    s = _join_state(case, g, author, by_rank, m, store.handle)
    s["keep"] = store
    s["single"] = case["viewers"] == 1 and case["lookups"] == 1
    return s


def _doc_ids(items, seed):
    """Distinct document ids for item numbers: a bijection on [0, 2^62)."""
    mask = (1 << 62) - 1
    return ((items * 0x2545F4914F6CDD1D) & mask) ^ ((seed * 0x9E3779B97F4A7C15 + 12345) & mask)


def _index(docs, capacity, doc, m, seed, g):
    """An indexed store holding items [0, docs), built by one ingestion batch."""
    author, by_rank = _authors(docs, m, True, g)
    store = _Store(P.cc_store_create_indexed(capacity, doc))
    ws = torch.empty(P.cc_upsert_workspace_bytes(docs), dtype=torch.uint8, device=DEV)
    ids = _doc_ids(torch.arange(docs, device=DEV), seed)
    P.cc_store_upsert(store.handle, ids, author, _rows(docs, doc, g), ws)
    return store, author, by_rank


def _prepare_request(case, seed):
    g = _gen(seed, 0)
    m = max(1_000, case["docs"], 4 * case["k"])
    store, author, by_rank = _index(case["docs"], case["docs"], case["doc"], m, seed, g)
    s = _join_state(case, g, author, by_rank, m, store.handle)
    cand = s["cand"]
    absent = torch.rand(cand.numel(), device=DEV, generator=g) < case["miss"]
    s["ids"] = _doc_ids(torch.where(absent, cand + case["docs"], cand), seed)
    s["cand"] = torch.empty_like(cand)          # the positions, written by each pass
    s["keep"] = store
    s["single"] = case["viewers"] == 1
    return s


def _prepare_sort(case, seed):
    g = _gen(seed, 0)
    ks = _sizes(case["k_lo"], case["k"], case["viewers"], 2)
    m = max(case["ids"], 4 * case["k"])
    keys = torch.cat([_unique(m, k, g) for k in ks])
    total = keys.numel()
    ws = P.cc_sort_workspace_bytes(total, len(ks))
    rows = _rows(total, case["row"], g)
    return {"kind": "sort", "offsets": _offsets(ks), "keys": keys, "rows": rows,
            "keys_out": torch.empty_like(keys), "rows_out": torch.empty_like(rows),
            "workspace": torch.empty(ws, dtype=torch.uint8, device=DEV),
            "max_keys": max(ks) if case["bound"] else 0,
            "key_bits": (m - 1).bit_length() if case["bits"] else 0}


def _prepare_ingest(case, seed):
    g = _gen(seed, 0)
    docs, n = case["docs"], case["n"]
    m = max(1_000, docs)
    store, author, by_rank = _index(docs, docs + n, case["doc"], m, seed, g)
    n_new = int(n * case["new"])
    items = torch.cat([torch.arange(docs, docs + n_new, device=DEV),
                       torch.randint(0, docs, (n - n_new,), device=DEV, generator=g)])
    rep = torch.rand(n, device=DEV, generator=g) < case["repeat"]
    items = torch.where(rep, items[torch.randint(0, n, (n,), device=DEV, generator=g)], items)
    items = items[torch.randperm(n, device=DEV, generator=g)]
    keys = _keys(1_000, m, by_rank, g)
    return {"kind": "ingest", "keep": store, "store": store.handle, "ids": _doc_ids(items, seed),
            "author": torch.randint(0, m, (n,), device=DEV, generator=g),
            "rows": _rows(n, case["doc"], g),
            "workspace": torch.empty(P.cc_upsert_workspace_bytes(n), dtype=torch.uint8, device=DEV),
            "pos": torch.empty(n, dtype=torch.int64, device=DEV), "keys": keys,
            "edge": _rows(1_000, 16, g),
            "out": torch.empty(n, case["doc"] + 16, dtype=torch.uint8, device=DEV),
            "hit": torch.empty(n, dtype=torch.int8, device=DEV)}


_PREPARE = {"join": _prepare_join, "padded": _prepare_join, "request": _prepare_request,
            "sort": _prepare_sort, "ingest": _prepare_ingest}


# ---- one pass -------------------------------------------------------------------------------

def _run_join(s):
    if s["single"]:
        P.cc_join(s["store"], s["cand"], s["keys"], s["edge"], s["out"], s["hit"],
                  default_row=s["default"])
    else:
        P.cc_join_batched(s["store"], s["cand_offsets"], s["cand"], s["key_offsets"], s["keys"],
                          s["edge"], s["out"], s["hit"], default_row=s["default"],
                          extra_keys=s["actor"], author_ids=s["authors"])
    return {"out": s["out"].view(torch.int64), "hit": s["hit"]}


def _run_padded(s):
    P.cc_join_batched_padded(s["store"], s["cand_offsets"], s["cand"], s["key_offsets"],
                             s["keys"], s["edge"], s["n_max"], s["out"], s["hit"], s["valid"],
                             default_row=s["default"], extra_keys=s["actor"])
    return {"out": s["out"].view(torch.int64), "hit": s["hit"], "valid": s["valid"]}


def _run_request(s):
    P.cc_resolve_ids(s["store"], s["ids"], s["cand"])
    return dict(_run_join(s), pos=s["cand"])


def _run_sort(s):
    P.cc_sort_affinity(s["offsets"], s["keys"], s["rows"], s["keys_out"], s["rows_out"],
                       s["workspace"], max_keys=s["max_keys"], key_bits=s["key_bits"])
    return {"keys": s["keys_out"], "rows": s["rows_out"].view(torch.int64)}


def _run_ingest(s):
    new, rejected = P.cc_store_upsert(s["store"], s["ids"], s["author"], s["rows"],
                                      s["workspace"])
    P.cc_resolve_ids(s["store"], s["ids"], s["pos"])
    P.cc_join(s["store"], s["pos"], s["keys"], s["edge"], s["out"], s["hit"])
    return {"new": new, "rejected": rejected, "pos": s["pos"], "hit": s["hit"],
            "out": s["out"].view(torch.int64)}


_RUN = {"join": _run_join, "padded": _run_padded, "request": _run_request, "sort": _run_sort,
        "ingest": _run_ingest}


def run(s):
    return _RUN[s["kind"]](s)
