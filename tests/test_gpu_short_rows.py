"""Summaries of short rows (at most 256 sixteen-byte units): 4 to 64 lanes share a row, a wavefront takes up to
16 rows a step and hands over 64 rows' totals at a time.  Row lengths at the edges of the lane counts, row
counts at the edges of steps, of hand-overs and of wavefronts, requests without rows, keep vectors, bad
indexes, rows with infinities and NaN, dense and paged; tolerances as in _util (absmax exact, norms 1e-3,
means against mean|x|)."""
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


def _one(B, x, reqs, out, mask, keep=None, index=None, **how):
    """The record of one observe, from the ring."""
    s = torch.cuda.current_stream().cuda_stream
    with B.Ring(64 << 20, 64 << 20, max_reqs_per_observe=4096) as ring:
        ring.debug_fill_rings(0xA5)
        km = None if keep is None else torch.from_numpy(np.asarray(keep, dtype=np.uint8)).to(DEV)
        if how:
            ring.observe_paged(5, x, how["table"], reqs, block_size=how["block"], n_heads=x.shape[2], head_dim=x.shape[3],
                               heads_sel=how["heads"], step_id=3, stream=s, out_dtype=out, summary_mask=mask, keep_mask=km)
        else:
            ri = None if index is None else torch.from_numpy(np.asarray(index, dtype=np.int32)).to(DEV)
            ring.observe_tensor(5, x, reqs, step_id=3, stream=s, out_dtype=out, summary_mask=mask, keep_mask=km, row_index=ri)
        ring.drain(B.DRAIN_FLUSH)
        (v,) = ring.poll_host()
        return v.bytes(), ring.get_stats().bad_rows


def _ragged(counts, rng):
    base, reqs = 0, []
    for i, n in enumerate(counts):
        step = int(rng.integers(1, 4))
        reqs.append((10 + i, base, int(rng.integers(0, 3)), int(n), step))
        base += 3 + max(1, int(n)) * step
    return np.array(reqs, dtype=np.uint32), base


@pytest.mark.parametrize("units", [1, 2, 4, 15, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("dtype,out,mask", [("bf16", 0, 7), ("bf16", 4, 5), ("fp16", 2, 2), ("fp32", 3, 7)])
def test_dense_ragged(B, units, dtype, out, mask):
    td = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[dtype]
    elems = units * (4 if dtype == "fp32" else 8)
    rng = np.random.default_rng(units)
    # more than 1024 rows (or a keep vector): the general kernel; requests without rows in between
    counts = [0, 1, 63, 64, 65, 0, 0, 127, 640, 1, 200, 0]
    reqs, rows = _ragged(counts, rng)
    x = prng.randn_bf16(units, rows * elems, DEV).view(rows, elems).to(td)
    x[5, 0], x[70, elems - 1] = float("inf"), float("nan")
    for keep in (None, rng.integers(0, 2, len(counts)), np.zeros(len(counts), np.uint8)):
        got, bad = _one(B, x, reqs, out, mask, keep=keep)
        ref = orc.build_record(x.cpu(), reqs, seq=0, step_id=3, point_id=5, out_dtype=out, summary_mask=mask, keep_mask=keep)
        at = np.concatenate([np.arange(n) * s + b + t for (_, b, t, n, s), k in
                             zip(reqs.tolist(), np.ones(len(counts)) if keep is None else keep) if k] or [[]]).astype(int)
        mean_abs = x.float().abs().mean(1).cpu().numpy()[at]
        compare_record(got, ref, what=f"{units} {dtype} {out} {mask} {keep}", mean_abs=mean_abs)
        assert bad == 0


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 2047, 2048, 2049])
def test_row_counts_and_bad_indexes(B, n):
    x = prng.randn_bf16(n, 500 * 256, DEV).view(500, 256)
    rng = np.random.default_rng(n)
    index = rng.integers(0, 500, n).astype(np.int32)
    index[::5] = np.array([-1, 500, 2 ** 31 - 1, -2 ** 31])[np.arange(len(index[::5])) % 4]
    reqs = np.array([[1, 0, 0, n, 1]], dtype=np.uint32)
    keep = [1]                                              # the general kernel also for few rows
    got, bad = _one(B, x, reqs, 1, 5, keep=keep, index=index)
    assert bad == len(index[::5])
    y = torch.cat([x.cpu(), torch.zeros(1, 256, dtype=torch.bfloat16)])
    fixed = np.where((index < 0) | (index >= 500), 500, index).astype(np.int32)
    ref = orc.build_record(y, reqs, seq=0, step_id=3, point_id=5, out_dtype=1, summary_mask=5, keep_mask=keep, row_index=fixed)
    compare_record(got, ref, what=str(n))


@pytest.mark.parametrize("heads,dim,out", [([1], 64, 0), ([0, 3], 128, 1), ([0, 1, 2], 80, 0), ([3, 0, 1, 2], 256, 4), ([2], 8, 1)])
def test_paged(B, heads, dim, out):
    blocks, block, n_heads, seqs = 40, 16, 4, 5
    x = prng.randn_bf16(dim, blocks * block * n_heads * dim, DEV).view(blocks, block, n_heads, dim)
    table = torch.from_numpy(prng.permutation(3, blocks).astype(np.int32).reshape(seqs, -1))
    reqs = np.array([[7, 1, 0, 100, 1], [8, 4, 3, 40, 3], [9, 0, 127, 1, 1], [10, 2, 5, 0, 1], [11, 3, 0, 128, 1]], dtype=np.uint32)
    got, _ = _one(B, x, reqs, out, 7, table=table.to(DEV), block=block, heads=heads)
    spec = configs.PagedSpec(block, n_heads, dim, heads, table)
    ref = orc.build_record(x.cpu(), reqs, seq=0, step_id=3, point_id=5, out_dtype=out, summary_mask=7, paged=spec)
    compare_record(got, ref, what=f"{heads} {dim}")


@pytest.mark.parametrize("units", [3, 32, 96, 200, 256])
def test_batched_summaries_have_the_bits_of_single_ones(B, units):
    """9 x 1000 rows in one launch take the general kernel, 1000 rows alone the decode-shaped one."""
    xs = [prng.randn_bf16(100 + i, 1000 * units * 8, DEV).view(1000, units * 8) for i in range(9)]
    reqs = np.array([[i, i, 0, 1, 1] for i in range(1000)], dtype=np.uint32)
    s = torch.cuda.current_stream().cuda_stream
    got = []
    for batched in (True, False):
        with B.Ring(256 << 20, 256 << 20, max_reqs_per_observe=1024) as ring:
            if batched:
                ring.observe_batch(range(9), xs, reqs, step_id=1, stream=s, out_dtype=1, summary_mask=7)
            else:
                for p, x in enumerate(xs):
                    ring.observe_tensor(p, x, reqs, step_id=1, stream=s, out_dtype=1, summary_mask=7)
            ring.drain(B.DRAIN_FLUSH)
            got.append([v.bytes() for v in ring.poll_host()])
    assert len(got[0]) == len(got[1]) == 9
    for a, b in zip(*got):
        assert np.array_equal(a, b)
