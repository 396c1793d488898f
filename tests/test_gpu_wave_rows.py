"""Summaries of rows of more than 256 units with a wavefront per row (launches of 2048 rows and more): row lengths at
the edges of its two to four parts, ragged rows with requests that have none, keep vectors, bad indexes, rows off
the 16-byte grid, paged rows, one or two rows per wavefront, infinities and NaN; against the oracle (tolerances as in
_util), and bit for bit against the decode-shaped kernel and the workgroup-per-row path."""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import configs, prng
from _util import compare_record

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


def _record(B, observe):
    with B.Ring(256 << 20, 256 << 20, max_reqs_per_observe=4096) as ring:
        ring.debug_fill_rings(0xA5)
        observe(ring, torch.cuda.current_stream().cuda_stream)
        ring.drain(B.DRAIN_FLUSH)
        views = ring.poll_host()
        return [v.bytes() for v in views], ring.get_stats().bad_rows


@pytest.mark.parametrize("elems,lead", [(2056, 0), (3072, 0), (4096, 0), (4104, 0), (5120, 0), (6144, 0), (2057, 1), (4097, 0), (6100, 3)])
@pytest.mark.parametrize("dtype,out,mask", [("bf16", 0, 7), ("bf16", 4, 5), ("fp16", 2, 1), ("fp32", 0, 7)])
@pytest.mark.parametrize("rows", [2048, 4101])
def test_dense_ragged(B, elems, lead, dtype, out, mask, rows):
    if dtype == "fp32":
        elems, lead = elems // 2, 0
    n_src = 500
    td = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[dtype]
    x = prng.randn_bf16(elems, n_src * (elems + lead), DEV).view(n_src, elems + lead)[:, lead:].to(td)
    if dtype == "bf16" and lead:
        assert not x.is_contiguous()
    x[3, 1], x[4, elems - 1] = float("inf"), float("nan")
    rng = np.random.default_rng(elems)
    counts = [0, 1, rows - 700, 0, 63, 600, 36, 0]
    assert sum(counts) == rows
    reqs = np.array([[i, 0, 0, c, 1] for i, c in enumerate(counts)], dtype=np.uint32)
    index = rng.integers(0, n_src, rows).astype(np.int32)
    index[::311] = n_src
    for keep in (None, np.array([1, 1, 1, 0, 0, 1, 1, 1], dtype=np.uint8)):
        km = None if keep is None else torch.from_numpy(keep).to(DEV)
        (got,), bad = _record(B, lambda ring, s: ring.observe_tensor(
            6, x, reqs, step_id=2, stream=s, out_dtype=out, summary_mask=mask, keep_mask=km,
            row_index=torch.from_numpy(index).to(DEV)))
        kept = np.ones(rows, bool) if keep is None else np.concatenate([np.full(c, k) for c, k in zip(counts, keep)]).astype(bool)
        assert bad == int(((index == n_src) & kept).sum())
        y = torch.cat([x.cpu(), torch.zeros(1, elems, dtype=td)])
        ref = orc.build_record(y, reqs, seq=0, step_id=2, point_id=6, out_dtype=out, summary_mask=mask, keep_mask=keep, row_index=index)
        compare_record(got, ref, what=f"{elems} {dtype}", mean_abs=y.float().abs().mean(1).numpy()[index[kept]])


@pytest.mark.parametrize("heads,dim,out", [([0, 2, 1], 704, 0), ([1, 0], 1100, 1), ([2, 1, 0], 701, 0)])
def test_paged(B, heads, dim, out):
    blocks, block, n_heads, seqs = 160, 16, 3, 4
    x = prng.randn_bf16(dim, blocks * block * n_heads * dim, DEV).view(blocks, block, n_heads, dim)
    table = torch.from_numpy(prng.permutation(5, blocks).astype(np.int32).reshape(seqs, -1))
    reqs = np.array([[7, 1, 0, 640, 1], [8, 3, 3, 500, 1], [9, 0, 0, 0, 1], [11, 2, 0, 640, 1], [12, 0, 5, 400, 1]], dtype=np.uint32)
    (got,), _ = _record(B, lambda ring, s: ring.observe_paged(
        1, x, table.to(DEV), reqs, block_size=block, n_heads=n_heads, head_dim=dim, heads_sel=heads, step_id=2, stream=s,
        out_dtype=out, summary_mask=5))
    ref = orc.build_record(x.cpu(), reqs, seq=0, step_id=2, point_id=1, out_dtype=out, summary_mask=5,
                           paged=configs.PagedSpec(block, n_heads, dim, heads, table))
    compare_record(got, ref, what=f"{heads} {dim}")


@pytest.mark.parametrize("units", [257, 384, 512, 513, 700, 768, 769, 1024, 1500])
@pytest.mark.parametrize("out", [0, 1])
def test_batches_have_the_bits_of_single_records(B, units, out):
    """17 x 1000 rows in one launch, and 1000 rows alone (decode-shaped, or a workgroup per row)."""
    x = prng.randn_bf16(units, 1100 * units * 8, DEV).view(1100, units * 8)
    xs = [x[5 * i:5 * i + 1000] for i in range(17)]
    reqs = np.array([[i, i, 0, 1, 1] for i in range(1000)], dtype=np.uint32)
    n = 17 if out == 0 else 5
    reqs = reqs if out == 0 else reqs[:500]
    how = dict(step_id=1, out_dtype=out, summary_mask=7)
    one = [_record(B, lambda ring, s, p=p: ring.observe_tensor(p, xs[p], reqs, stream=s, **how))[0][0]
           for p in range(n)]
    many, _ = _record(B, lambda ring, s: ring.observe_batch(range(n), xs[:n], reqs, stream=s, **how))
    for a, b in zip(many, one):
        assert np.array_equal(a[:8], b[:8]) and np.array_equal(a[16:], b[16:])       # (all but the sequence number)
