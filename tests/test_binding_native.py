"""The native marshalling of observe_into and of prepared observes hands the C ABI what the Python functions do, and what
it does not take itself comes back to them with the same results and errors."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2605_11093_amd import binding as B

native = pytest.importorskip("paper_2605_11093_amd._dmi_python")
INTO = C.CFUNCTYPE(C.c_int32, C.c_uint32, C.c_void_p, C.c_void_p, C.c_void_p, C.c_uint64, C.c_uint64, C.c_uint32, C.c_void_p,
                   C.c_uint64, C.c_void_p, C.c_void_p)


class Sub(torch.Tensor):
    pass


@pytest.fixture
def seen(monkeypatch):
    """Calls as the entry point sees them: (how, arguments)."""
    calls, code = [], [0]

    def note(how, point, t, sel, xf, seq, step, rank, out, out_bytes, n, stream):
        t, sel, xf = (k.from_buffer_copy(C.string_at(p, C.sizeof(k)) if isinstance(p, int) else p)
                      for k, p in ((B.Tensor, t), (B.Selection, sel), (B.Transform, xf)))
        reqs = C.string_at(sel.reqs, 20 * sel.n_reqs) if sel.n_reqs else b""
        calls.append((how, point, t.data, t.dtype, list(t.shape), list(t.stride), sel.n_reqs, reqs, sel.keep_mask_dev,
                      sel.row_index_dev, xf.out_dtype, xf.summary_mask, seq, step, rank, out, out_bytes, stream))
        C.cast(n, C.POINTER(C.c_uint64))[0] = 77
        return code[0]

    fn = INTO(lambda *a: note("native", *a))
    B.lib()
    native.bind_into(C.cast(fn, C.c_void_p).value)
    general = lambda *a: note("general", *a)        # noqa: E731
    yield calls, code, general
    native.bind_into(C.cast(B.lib().dmi_observe_into, C.c_void_p).value)


X = torch.zeros(7, 40, dtype=torch.float16)[:, 3:35]
REQS = np.array([[1, 2, 3, 4, 5], [6, 7, 8, 9, 10]], dtype=np.uint32)
OUT = torch.zeros(64, dtype=torch.int32)
KEEP, INDEX = torch.ones(2, dtype=torch.uint8), torch.zeros(4, dtype=torch.int32)
PLAIN = {
    "all": ((9, X, REQS, OUT), dict(seq=5, step_id=6, rank_tag=2, out_dtype=4, summary_mask=3, keep_mask=KEEP, row_index=INDEX, stream=11)),
    "few": ((9, X, REQS, OUT), dict(seq=5, step_id=6)),
    "names": ((), dict(stream=3, step_id=1, seq=2, out=OUT, reqs=REQS, tensor=X.float(), point_id=4)),
    "wraps": ((-1, X.bfloat16(), REQS, OUT), dict(seq=-1, step_id=2**64 + 5, rank_tag=-2, summary_mask=-1, out_dtype=None, keep_mask=None)),
    "no requests": ((1, X, REQS[:0], OUT), dict(seq=0, step_id=0, out_dtype=0, stream=0)),
    "read-only": ((1, X, np.frombuffer(REQS.tobytes(), dtype=np.uint32).reshape(2, 5), OUT), dict(seq=0, step_id=0)),
    "bool": ((True, X, REQS, OUT), dict(seq=True, step_id=0)),
}
OTHER = {
    "list": ((1, X, REQS.tolist(), OUT), dict(seq=0, step_id=0)),
    "int64": ((1, X, REQS.astype(np.int64), OUT), dict(seq=0, step_id=0)),
    "columns": ((1, X, np.asfortranarray(REQS), OUT), dict(seq=0, step_id=0)),
    "flat": ((1, X, REQS.reshape(-1), OUT), dict(seq=0, step_id=0)),
    "vector": ((1, X[0], REQS, OUT), dict(seq=0, step_id=0)),
    "subclass": ((1, X.as_subclass(Sub), REQS, OUT), dict(seq=0, step_id=0)),
    "numpy mask": ((1, X, REQS, OUT), dict(seq=0, step_id=0, summary_mask=np.int64(3), out_dtype=np.int64(1))),
    "no stream": ((1, X, REQS, OUT), dict(seq=0, step_id=0, stream=None)),
}
WRONG = {
    "missing": ((1, X, REQS, OUT), dict(seq=0)),
    "unknown": ((1, X, REQS, OUT), dict(seq=0, step_id=0, what=1)),
    "twice": ((1, X, REQS, OUT), dict(seq=0, step_id=0, out=OUT)),
    "too many": ((1, X, REQS, OUT, 5), dict(seq=0, step_id=0)),
    "dtype": ((1, X.int(), REQS, OUT), dict(seq=0, step_id=0)),
    "cube": ((1, X.contiguous().view(7, 4, 8), REQS, OUT), dict(seq=0, step_id=0)),
    "float": ((1, X, REQS, OUT), dict(seq=0.5, step_id=0)),
    "tensor": ((1, None, REQS, OUT), dict(seq=0, step_id=0)),
    "storage": ((1, X.to_sparse(), REQS, OUT), dict(seq=0, step_id=0)),
}


@pytest.mark.parametrize("name", [*PLAIN, *OTHER])
def test_same_arguments(seen, monkeypatch, name):
    calls, _, general = seen
    args, kw = {**PLAIN, **OTHER}[name]
    if name in PLAIN:
        assert B.observe_into(*args, **kw) == 77
    with monkeypatch.context() as m:
        m.setattr(B, "_into_fn", general)
        assert B.observe_into(*args, **kw) == 77
    if name in OTHER:
        assert [c[0] for c in calls] == ["general"]
        return
    assert [c[0] for c in calls] == ["native", "general"]
    a, b = calls
    mask = {1: 2**32 - 1, 12: 2**64 - 1, 13: 2**64 - 1, 14: 2**32 - 1}      # (ctypes takes an int's low bits)
    for i, (p, q) in enumerate(zip(a[1:], b[1:]), 1):
        if i in mask:
            q = int(q) & mask[i]
        assert (p or 0) == (q or 0), i


@pytest.mark.parametrize("name", [*WRONG])
def test_same_errors(seen, monkeypatch, name):
    calls, _, general = seen
    args, kw = WRONG[name]
    with pytest.raises(Exception) as a:
        B.observe_into(*args, **kw)
    assert not calls
    with monkeypatch.context() as m:
        m.setattr(B, "_into_fn", general)
        if name == "float":                         # (a stand-in does not convert; the entry point refuses it)
            assert a.type is C.ArgumentError
            return
        with pytest.raises(Exception) as b:
            B.observe_into(*args, **kw)
    assert a.type is b.type and str(a.value) == str(b.value)


def test_status_codes(seen):
    calls, code, _ = seen
    code[0] = B.ERR_TOO_LARGE
    with pytest.raises(B.DmiError) as e:
        B.observe_into(1, X, REQS, OUT, seq=0, step_id=0)
    assert e.value.code == B.ERR_TOO_LARGE
    assert B.observe_into(1, X, REQS, OUT, seq=0, step_id=0, allow=(B.ERR_TOO_LARGE,)) == 77
    assert len(calls) == 2


def test_prepared_observe():
    got = []
    fn = C.CFUNCTYPE(C.c_int32, C.c_void_p, C.c_uint32, C.c_void_p, C.c_void_p, C.c_void_p, C.c_uint64, C.c_void_p)(
        lambda *a: got.append(a) or -5)

    class P(native.Prepared):
        def _call(self, step_id, stream):
            return ("python", step_id, stream)

    p = P()
    assert p(1, 2) == ("python", 1, 2)              # not bound
    p._bind(C.cast(fn, C.c_void_p).value, 0x1000, 7, 0x2000, 0x3000, 0x4000)
    assert p(9, 0) == -5 and p(2**64 + 3, 0x50) == -5
    assert got == [(0x1000, 7, 0x2000, 0x3000, 0x4000, 9, None), (0x1000, 7, 0x2000, 0x3000, 0x4000, 3, 0x50)]
    assert p(step_id=1, stream=2) == ("python", 1, 2) and p(1, None) == ("python", 1, None) and p(1.5, 2) == ("python", 1.5, 2)
    with pytest.raises(TypeError):
        p(1)
    assert len(got) == 2
