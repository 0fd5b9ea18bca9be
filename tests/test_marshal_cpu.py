"""The binding's native marshalling (csrc/marshal.c) on the CPU: host tensors that report GPU
residency, and C functions that record their arguments, stand in for the tensors and the library. Every
call is made once with the native path in front and once through binding.py's checks alone; both
must reach the same C function with the same arguments, or raise the same error."""
import ctypes
import subprocess
import sys
import textwrap

import pytest
import torch

import paper_2609_22441_amd.binding as B

DOC, EDGE = 32, 16
HOT = ("cc_join", "cc_join_batched", "cc_join_batched_authors", "cc_join_batched_padded",
       "cc_resolve_ids", "cc_sort_affinity", "cc_sort_affinity_method", "cc_store_upsert")


class OnGpu:
    """A host tensor that reports GPU residency."""
    is_cuda = True

    def __init__(self, t):
        self.t = t

    def __getattr__(self, k):
        return getattr(self.t, k)


class Off:
    """A marshal module that answers None to everything."""
    def __getattr__(self, name):
        return lambda *a: None


class Recorder:
    """Functions with the library's signatures that record (name, arguments) and return 0; as
    attributes for ctypes callers, and their addresses (at_*) for the native path."""

    def __init__(self, real, marshal):
        self.calls, self.keep, self.asked = [], [], 0
        self.marshal = marshal
        for name in HOT + ("cc_store_info",):
            f = ctypes.CFUNCTYPE(ctypes.c_int, *getattr(real, name).argtypes)(
                self._info if name == "cc_store_info" else self._record(name))
            self.keep.append(f)
            setattr(self, name, f)
            setattr(self, "at_" + name, ctypes.cast(f, ctypes.c_void_p).value)

    def _info(self, store, n, width):
        self.asked += 1
        if width:
            width[0] = DOC
        return 0

    def _record(self, name):
        def call(*args):
            # Pointers to pointers: the pointers themselves; pointers to results: left out.
            self.calls.append((name, [(a[0] if a else None) if isinstance(a, ctypes.POINTER(ctypes.c_void_p))
                                      else a for a in args if not isinstance(a, ctypes.POINTER(ctypes.c_int64))]))
            return 0
        return call


@pytest.fixture
def both(monkeypatch):
    """both(call) runs call(binding) on each path and returns the two outcomes."""
    from paper_2609_22441_amd import _marshal
    real = B.lib()
    _marshal.init(OnGpu, torch.int64, torch.int8, lambda: 7)
    monkeypatch.setattr(B, "_current_stream", lambda: 7)

    def run(call):
        got = []
        for marshal in (_marshal, Off()):
            rec = Recorder(real, marshal)
            monkeypatch.setattr(B, "_lib", rec)
            try:
                call()
                got.append(rec.calls)
            except Exception as e:
                got.append((type(e), str(e), rec.calls))
        return got

    yield run
    _marshal.init(torch.Tensor, torch.int64, torch.int8, B._current_stream)


def g(*shape, dtype=torch.int64):
    return OnGpu(torch.zeros(*shape, dtype=dtype))


N, K, V = 10, 6, 2


def batch(L=2):
    return dict(cand_offsets=g(V + 1), cand_idx=g(N), key_offsets=g(V + 1), edge_keys=g(K),
                edge_feats=g(K, EDGE, dtype=torch.uint8),
                out=g(N, DOC + L * EDGE, dtype=torch.uint8), hit_mask=g(N, L, dtype=torch.int8))


def padded(L=2, n_max=5):
    s = V * n_max
    return dict(batch(L), out=g(s, DOC + L * EDGE, dtype=torch.uint8),
                hit_mask=g(s, L, dtype=torch.int8), valid_mask=g(s, dtype=torch.int8), n_max=n_max)


def same(got):
    assert got[0] == got[1]
    return got[0]


# What may stand for the second lookup's keys. None in a list is no list of keys: it raises, and is
# not taken for a call with one lookup.
EXTRA = {"one": lambda: [g(N)], "tuple": lambda: (g(N),), "set": lambda: {g(N)}, "none": lambda: None,
         "empty": lambda: [], "a list of None": lambda: [None], "a tuple of None": lambda: (None,),
         "two": lambda: [g(N), g(N)], "short": lambda: [g(N - 1)], "32 bits": lambda: [g(N, dtype=torch.int32)]}


@pytest.mark.parametrize("kind", EXTRA)
def test_second_lookup(both, kind):
    extra = EXTRA[kind]()
    L = 1 + (len(extra) if extra else 0)
    for form, args in ((B.cc_join_batched, batch(max(L, 2))), (B.cc_join_batched_padded, padded(max(L, 2)))):
        got = same(both(lambda: form(1, extra_keys=extra, stream=0, **args)))
        if kind in ("a list of None", "a tuple of None"):
            assert got[0] is ValueError and got[2] == []
        elif kind in ("short", "32 bits"):
            assert got[0] in (ValueError, TypeError) and got[2] == []
        else:
            assert len(got) == 1 and (L if L < 3 else 3) in got[0][1]


def test_plain_calls(both):
    """The other entry points and their options."""
    cand, ids, pos, ws, rows = g(N), g(N), g(N), g(64), g(N, DOC, dtype=torch.uint8)
    one = dict(edge_keys=g(K), edge_feats=g(K, EDGE, dtype=torch.uint8),
               out=g(N, DOC + EDGE + 8, dtype=torch.uint8), hit_mask=g(N, dtype=torch.int8))
    row, many = g(EDGE, dtype=torch.uint8), batch(1)
    sort = (g(V + 1), g(K), g(K, EDGE, dtype=torch.uint8), g(K), g(K, EDGE, dtype=torch.uint8), ws)
    for name, call in (("cc_join", lambda: B.cc_join(1, cand, **one)),
                       ("cc_join", lambda: B.cc_join(1, cand, default_row=row, stream=3, **one)),
                       ("cc_join_batched_authors", lambda: B.cc_join_batched(1, author_ids=ids, **many)),
                       ("cc_resolve_ids", lambda: B.cc_resolve_ids(1, ids, pos)),
                       ("cc_store_upsert", lambda: B.cc_store_upsert(1, ids, pos, rows, ws)),
                       ("cc_sort_affinity_method",
                        lambda: B.cc_sort_affinity(*sort, max_keys=5, method=2, key_bits=9))):
        got = same(both(call))
        assert len(got) == 1 and got[0][0] == name


@pytest.mark.parametrize("error", [KeyboardInterrupt, MemoryError, RuntimeError])
def test_an_exception_on_the_way_is_raised(both, monkeypatch, error):
    """An interrupt while the native path asks for the current stream is not lost, and nothing is
    called."""
    from paper_2609_22441_amd import _marshal
    raised = []

    def once():
        if not raised:
            raised.append(1)
            raise error("once")
        return 7

    _marshal.init(OnGpu, torch.int64, torch.int8, once)
    rec = Recorder(B.lib(), _marshal)
    monkeypatch.setattr(B, "_lib", rec)
    with pytest.raises(error, match="once"):
        B.cc_resolve_ids(1, g(N), g(N))
    assert rec.calls == []
    B.cc_resolve_ids(1, g(N), g(N))
    assert len(rec.calls) == 1


@pytest.mark.parametrize("error", [AttributeError, TypeError, OverflowError])
@pytest.mark.parametrize("name", ["numel", "is_contiguous", "data_ptr"])
def test_an_argument_without_a_tensors_methods_is_not_plain(both, name, error):
    class Odd(OnGpu):
        pass

    def fail(self):
        raise error("odd")

    from paper_2609_22441_amd import _marshal
    _marshal.init(Odd, torch.int64, torch.int8, lambda: 7)
    rec = Recorder(B.lib(), _marshal)
    x = Odd(torch.zeros(N, dtype=torch.int64))
    assert _marshal.resolve(rec.at_cc_resolve_ids, 1, x, x, 0) == 0 and len(rec.calls) == 1
    setattr(Odd, name, fail)
    assert _marshal.resolve(rec.at_cc_resolve_ids, 1, x, x, 0) is None and len(rec.calls) == 1


def test_a_refused_call_reads_no_store_handle(both):
    """The row width is asked of the store only when every argument that does not need it has passed:
    with one of those missing, the native path answers None without reading the handle."""
    from paper_2609_22441_amd import _marshal
    rec = Recorder(B.lib(), _marshal)
    info, b, p = rec.at_cc_store_info, batch(), padded()
    row = g(EDGE, dtype=torch.uint8)
    head = [b[k] for k in ("cand_offsets", "cand_idx", "key_offsets", "edge_keys", "edge_feats")]
    # (function, arguments, place of the output rows: the one argument checked against the width)
    calls = [
        (_marshal.join, [rec.at_cc_join, info, 1, g(N), g(K), b["edge_feats"],
                         g(N, DOC + EDGE, dtype=torch.uint8), g(N, dtype=torch.int8), row, 0], 6),
        (_marshal.batched, [rec.at_cc_join_batched, rec.at_cc_join_batched_authors, info, 1, *head,
                            row, g(N), 0, b["out"], b["hit_mask"], g(N)], 12),
        (_marshal.padded, [rec.at_cc_join_batched_padded, info, 1, *head, row, g(N), 0, p["n_max"],
                           p["out"], p["hit_mask"], p["valid_mask"]], 12),
        (_marshal.upsert, [rec.at_cc_store_upsert, info, 1, g(N), g(N), g(N, DOC, dtype=torch.uint8),
                           g(64), 0], None)]
    for call, args, out in calls:
        for i in range(args.index(1) + 1, len(args)):
            if i != out:
                assert call(*args[:i], "odd", *args[i + 1:]) is None
                assert rec.asked == 0 and rec.calls == [], (call.__name__, i)
        assert call(*args) in (0, (0, 0, 0)) and rec.asked == 1 and len(rec.calls) == 1
        rec.calls.clear()
        rec.asked = 0


def _python(code):
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(code)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stderr


def test_the_library_loads_without_torch_and_without_the_native_path():
    _python("""
        import sys
        sys.modules["torch"] = None
        sys.modules["paper_2609_22441_amd._marshal"] = None
        import paper_2609_22441_amd as P
        assert P.cc_sort_workspace_bytes(1000, 2) > 0 and P.cc_status_string(0)
        """)


def test_calls_without_the_native_path_are_checked_in_python():
    err = _python("""
        import sys
        sys.modules["paper_2609_22441_amd._marshal"] = None
        import torch
        import paper_2609_22441_amd as P
        x = torch.zeros(4, dtype=torch.int64)
        for n in (1, 2):
            try:
                P.cc_resolve_ids(1, x, x)
            except ValueError as e:
                assert "GPU memory" in str(e)
            else:
                raise SystemExit("no error")
        """)
    assert err.count("not built") == 1
