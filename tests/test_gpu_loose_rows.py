"""Rows that do not sit on a 16-byte grid: moved in 16-byte units at any address when they have at least 16 bytes
(the last unit of a row or of a head overlaps the one in front of it), element by element when they are
shorter.  Row lengths and offsets around the unit, around the work items of every path, records that wrap the ring
at every offset; against the oracle, bit-exact except the fp32 summaries (_util)."""
import numpy as np
import pytest
import torch

from oracle.stream import POLICY_BLOCK  # noqa: F401  (the helper's ring model)
import oracle as orc
from workloads import configs, prng
from _util import compare_record, compare_streams
from test_gpu_paths import _stream_through_small_ring

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


def _tensor(seed, rows, elems, lead, dtype):
    x = prng.randn_bf16(seed, rows * (elems + lead + 3), DEV).view(rows, elems + lead + 3)
    return x.to({"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[dtype])[:, lead:lead + elems]


@pytest.mark.parametrize("elems", [1, 3, 4, 7, 8, 9, 15, 16, 17, 23, 101, 255, 513, 2047, 2048, 2049, 2055, 4097, 8191, 8200])
@pytest.mark.parametrize("dtype,out,mask", [("bf16", 1, 0), ("bf16", 4, 0), ("bf16", 2, 5), ("bf16", 1, 7), ("bf16", 4, 1),
                                            ("fp16", 2, 0), ("fp16", 2, 7), ("fp32", 3, 0), ("fp32", 3, 7)])
def test_wrapping_streams(B, elems, dtype, out, mask):
    rows = 40
    xs = [_tensor(31 * elems + k, rows, elems, lead, dtype) for k, lead in enumerate((0, 1, 5))]
    reqs = np.array([[1, 0, 1, 5, 2], [2, 12, 0, 0, 1], [3, 13, 0, 9, 3], [4, 39, 0, 1, 1]], dtype=np.uint32)
    size = B.record_bytes(4, 15, elems, out, mask)
    got, ref = _stream_through_small_ring(
        B, lambda i: (xs[i % 3], reqs, dict(out_dtype=out, summary_mask=mask), dict(out_dtype=out, summary_mask=mask)), 9, size)
    compare_streams(got, ref)


@pytest.mark.parametrize("elems,lead", [(8, 1), (33, 0), (100, 2), (2050, 1), (8205, 3), (16384, 1)])
@pytest.mark.parametrize("dtype,out,mask", [("bf16", 1, 0), ("bf16", 4, 7), ("bf16", 0, 7), ("fp32", 3, 5)])
def test_many_rows_keep_vectors_and_bad_indexes(B, elems, lead, dtype, out, mask):
    rows, n = 300, 1500
    x = _tensor(elems, rows, elems, lead, dtype)
    rng = np.random.default_rng(elems)
    counts = [0, 700, 1, 299, 0, 500]
    reqs = np.array([[i, 0, 0, c, 1] for i, c in enumerate(counts)], dtype=np.uint32)
    index = rng.integers(0, rows, n).astype(np.int32)
    index[::97] = -1
    index[5::211] = rows
    keep = np.array([1, 1, 0, 1, 1, 1], dtype=np.uint8)
    s = torch.cuda.current_stream().cuda_stream
    with B.Ring(128 << 20, 128 << 20) as ring:
        ring.debug_fill_rings(0xA5)
        ring.observe_tensor(2, x, reqs, step_id=4, stream=s, out_dtype=out, summary_mask=mask,
                            keep_mask=torch.from_numpy(keep).to(DEV), row_index=torch.from_numpy(index).to(DEV))
        ring.drain(B.DRAIN_FLUSH)
        (v,) = ring.poll_host()
        got, bad = v.bytes(), ring.get_stats().bad_rows
    kept = np.concatenate([np.full(c, k) for c, k in zip(counts, keep)]).astype(bool)
    off = (index < 0) | (index >= rows)
    assert bad == int((off & kept).sum())
    y = torch.cat([x.cpu(), torch.zeros(1, elems, dtype=x.dtype)])
    fixed = np.where(off, rows, index).astype(np.int32)
    ref = orc.build_record(y, reqs, seq=0, step_id=4, point_id=2, out_dtype=out, summary_mask=mask, keep_mask=keep, row_index=fixed)
    compare_record(got, ref, what=f"{elems} {lead} {dtype}", mean_abs=y.float().abs().mean(1).numpy()[fixed[kept]])


@pytest.mark.parametrize("heads,dim", [([1], 8), ([0, 2], 12), ([2, 0, 1], 20), ([1, 2], 7), ([0, 1, 2], 129), ([0, 1, 2], 700)])
@pytest.mark.parametrize("dtype,out,mask", [("bf16", 1, 0), ("bf16", 4, 5), ("fp32", 3, 7)])
def test_paged(B, heads, dim, dtype, out, mask):
    blocks, block, n_heads, seqs = 20, 16, 3, 4
    x = _tensor(dim, blocks * block * n_heads, dim, 1, dtype)
    x = x.as_strided((blocks, block, n_heads, dim), (block * n_heads * (dim + 4), n_heads * (dim + 4), dim + 4, 1), x.storage_offset())
    table = torch.from_numpy(prng.permutation(3, blocks).astype(np.int32).reshape(seqs, -1))
    reqs = np.array([[7, 1, 0, 70, 1], [8, 3, 3, 20, 3], [9, 0, 79, 1, 1], [11, 2, 0, 80, 1]], dtype=np.uint32)
    spec = configs.PagedSpec(block, n_heads, dim, heads, table.to(DEV))
    size = B.record_bytes(4, 171, dim * len(heads), out, mask)
    kw = dict(out_dtype=out, summary_mask=mask)
    got, ref = _stream_through_small_ring(B, lambda i: (x, reqs, kw, kw), 4, size, paged=spec)
    compare_streams(got, ref)
