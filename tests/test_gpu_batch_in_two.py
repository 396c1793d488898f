"""Batches that go by two launches so that a flush can copy what the first has captured while the second runs: the stream of
records that the same tensors give when they are observed one by one (which other tests hold against the oracle), through several
flushes, and a record behind the cut against the oracle's.  (That these batches are cut, and where, is asserted on the CPU:
where_the_batches_of_the_gpu_test_are_cut in cpu_runtime/flush_rules_driver.cpp.)"""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import configs, prng

from _util import compare_record

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# tensors, requests, rows of each, width, source; statistics alone
CASES = [(4, 32, 2048, 1024, torch.float32, 7),     # capture_rows_kernel; three tensors, then one
         (4, 65, 3001, 128, torch.bfloat16, 7),     # the general kernel, short rows; one tensor, then three
         (4, 70, 930, 1024, torch.float32, 7)]      # the general kernel, longer ones; three, then one


@pytest.mark.parametrize("n,n_reqs,each,width,dtype,sums", CASES)
def test_dense(n, n_reqs, each, width, dtype, sums):
    from paper_2605_11093_amd import binding as B
    reqs = np.array([[70 + i, i * each, 0, each, 1] for i in range(n_reqs)], dtype=np.uint32)
    x = [torch.empty(n_reqs * each, width, dtype=dtype, device=DEV) for _ in range(n)]
    _both(B, x, reqs, 0, sums, None, lambda f, i, t: t.copy_(prng.randn_bf16(100 * f + i, t.numel(), DEV).view(t.shape)))


def test_paged():
    from paper_2605_11093_amd import binding as B
    block, heads, dim, per, n_reqs = 16, 4, 128, 256, 20
    g = torch.Generator(device=DEV).manual_seed(5)
    table = torch.randperm(n_reqs * per, generator=g, device=DEV).to(torch.int32).view(n_reqs, per)
    spec = configs.PagedSpec(block, heads, dim, [1, 2], table)
    reqs = np.array([[40 + i, i, 0, 4001, 1] for i in range(n_reqs)], dtype=np.uint32)
    x = [torch.empty(n_reqs * per, block, heads, dim, dtype=torch.bfloat16, device=DEV) for _ in range(8)]
    _both(B, x, reqs, 0, 5, spec, lambda f, i, t: t.copy_(prng.randn_bf16(100 * f + i, t.numel(), DEV).view(t.shape)))


def _both(B, x, reqs, out, sums, paged, fill):
    rows = int(reqs[:, 3].sum())
    elems = 256 if paged else x[0].shape[1]
    one = B.record_bytes(len(reqs), rows, elems, out, sums)
    ring_bytes = -(-5 * len(x) * one // 2 // 64) * 64           # a flush in three goes over the rings' ends
    s = torch.cuda.current_stream().cuda_stream
    kw = dict(stream=s, out_dtype=out, summary_mask=sums)
    with B.Ring(ring_bytes, ring_bytes, max_reqs_per_observe=128) as two, B.Ring(ring_bytes, ring_bytes, max_reqs_per_observe=128) as single:
        for flush in range(3):
            for i, t in enumerate(x):
                fill(flush, i, t)
            rc, done = two.observe_batch(range(len(x)), x, reqs, step_id=flush, paged=paged, **kw)
            assert rc == B.OK and done == len(x)
            two.drain(B.DRAIN_FLUSH)
            for p, t in enumerate(x):
                if paged:
                    single.observe_paged(p, t, paged.block_table, reqs, block_size=paged.block_size, n_heads=paged.n_heads,
                                         head_dim=paged.head_dim, heads_sel=paged.heads_sel, step_id=flush, **kw)
                else:
                    single.observe_tensor(p, t, reqs, step_id=flush, **kw)
            single.drain(B.DRAIN_FLUSH)
            a, b = two.poll_host(), single.poll_host()
            assert [v.seq for v in a] == [v.seq for v in b] == list(range(flush * len(x), (flush + 1) * len(x)))
            for p in range(len(x)):
                assert np.array_equal(a[p].bytes(), b[p].bytes()), (flush, p)
            if flush == 2 and paged is None:
                compare_record(a[-1].bytes(), orc.build_record(x[-1].cpu(), reqs, seq=a[-1].seq, step_id=flush, point_id=len(x) - 1,
                                                               out_dtype=out, summary_mask=sums))
            two.release_host(a[-1].seq)
            single.release_host(b[-1].seq)
        st = two.get_stats()
        assert st.captured_records == st.launched_records == 3 * len(x) and st.captured_bytes == st.drained_bytes == 3 * len(x) * one
