"""observe_into hands the C ABI the same structs, byte for byte, that the ctypes classes describe."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2605_11093_amd import binding as B


def _seen(monkeypatch, *args, code=0, **kw):
    got = {}

    def fake(point, t, sel, xf, seq, step, rank, out, out_bytes, n, stream):
        got.update(point=point, t=B.Tensor.from_buffer_copy(t), sel=B.Selection.from_buffer_copy(sel),
                   xf=B.Transform.from_buffer_copy(xf), rest=(seq, step, rank, out, out_bytes, stream))
        got["reqs"] = np.ctypeslib.as_array(C.cast(got["sel"].reqs, C.POINTER(C.c_uint32)), (got["sel"].n_reqs * 5,)).copy() \
            if got["sel"].n_reqs else np.zeros(0)
        C.cast(n, C.POINTER(C.c_uint64))[0] = 77
        return code
    monkeypatch.setattr(B, "_into_fn", fake)
    got["returned"] = B.observe_into(*args, **kw)
    return got


@pytest.mark.parametrize("reqs", [
    np.array([[1, 2, 3, 4, 5], [6, 7, 8, 9, 10]], dtype=np.uint32),
    [(1, 2, 3, 4, 5), (6, 7, 8, 9, 10)],
    np.array([[1, 2, 3, 4, 5], [6, 7, 8, 9, 10]], dtype=np.int64),
    np.array([[1, 6], [2, 7], [3, 8], [4, 9], [5, 10]], dtype=np.uint32).T,
    np.arange(1, 11, dtype=np.uint32),
    np.frombuffer(np.arange(1, 11, dtype=np.uint32).tobytes(), dtype=np.uint32).reshape(2, 5),     # read-only
])
def test_structs(monkeypatch, reqs):
    assert C.sizeof(B.Tensor) == 48 and C.sizeof(B.Selection) == 32 and C.sizeof(B.Transform) == 8
    x = torch.zeros(7, 40, dtype=torch.float16)[:, 3:35]
    keep, index, out = torch.ones(2, dtype=torch.uint8), torch.zeros(4, dtype=torch.int32), torch.zeros(256, dtype=torch.uint8)
    g = _seen(monkeypatch, 9, x, reqs, out, seq=5, step_id=6, rank_tag=2, summary_mask=3, keep_mask=keep, row_index=index, stream=11)
    assert g["returned"] == 77 and g["point"] == 9 and g["rest"] == (5, 6, 2, out.data_ptr(), 256, 11)
    assert (g["t"].data, g["t"].dtype, list(g["t"].shape), list(g["t"].stride)) == (x.data_ptr(), B.DT_FP16, [7, 32], [40, 1])
    assert (g["sel"].n_reqs, g["sel"].keep_mask_dev, g["sel"].row_index_dev) == (2, keep.data_ptr(), index.data_ptr())
    assert g["reqs"].tolist() == list(range(1, 11))
    assert (g["xf"].out_dtype, g["xf"].summary_mask) == (B.DT_FP16, 3)


def test_defaults_no_requests_and_errors(monkeypatch):
    x, out = torch.zeros(3, 8, dtype=torch.bfloat16), torch.zeros(64, dtype=torch.uint8)
    g = _seen(monkeypatch, 0, x, np.zeros((0, 5), np.uint32), out, seq=0, step_id=0, out_dtype=B.DT_NONE, summary_mask=-1)
    assert g["sel"].n_reqs == 0 and g["sel"].keep_mask_dev is None and g["sel"].row_index_dev is None and g["rest"][-1] is None
    assert (g["xf"].out_dtype, g["xf"].summary_mask) == (0, 0xFFFFFFFF)
    with pytest.raises(B.DmiError):
        _seen(monkeypatch, 0, x, [[0, 0, 0, 1, 1]], out, seq=0, step_id=0, code=B.ERR_TOO_LARGE)
    g = _seen(monkeypatch, 0, x, [[0, 0, 0, 1, 1]], out, seq=0, step_id=0, code=B.ERR_TOO_LARGE, allow=(B.ERR_TOO_LARGE,))
    assert g["returned"] == 77
    with pytest.raises(IndexError):
        B.observe_into(0, x.view(3, 2, 4), [[0, 0, 0, 1, 1]], out, seq=0, step_id=0)


def test_a_vector_is_handed_on_with_rows_of_length_zero(monkeypatch):
    out = torch.zeros(64, dtype=torch.uint8)
    g = _seen(monkeypatch, 0, torch.zeros(8, dtype=torch.bfloat16), [[0, 0, 0, 1, 1]], out, seq=0, step_id=0)
    assert list(g["t"].shape) == [8, 0] and list(g["t"].stride) == [1, 0]
