"""Rows that a launch deals flat: of 64 units and more in large launches, beside the same rows in a launch that is a little smaller and gives each a
wavefront: one row per request in a batch and ragged, raw, fp16 and fp8, on and off the 16-byte grid, with a keep vector, an
index and a record that wraps in the ring; shorter ones in batches of several sizes."""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import prng

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("elems", [512, 520, 517, 568])
@pytest.mark.parametrize("out", [1, 2, 4])
@pytest.mark.parametrize("how", ["plain", "keep", "index"])
def test_ragged(B, elems, out, how):
    s = torch.cuda.current_stream().cuda_stream
    for n_rows in (11900, 12100, 24400):
        x = prng.randn_bf16(n_rows, n_rows * elems, DEV).view(n_rows, elems)
        x[5, 3], x[7, elems - 1], x[n_rows - 1, 0] = float("nan"), float("inf"), -float("nan")
        each = n_rows // 50
        reqs = np.array([[i, each * i, 0, each - (i % 3), 1] for i in range(50)], dtype=np.uint32)
        keep = (np.arange(50) % 4 != 1).astype(np.uint8) if how == "keep" else None
        idx = np.random.default_rng(3).permutation(n_rows)[:int(reqs[:, 3].sum())].astype(np.int32) if how == "index" else None
        ref = orc.build_record(x.cpu(), reqs, seq=0, step_id=0, point_id=1, out_dtype=out, summary_mask=0, keep_mask=keep, row_index=idx)
        bound = B.record_bytes(50, int(reqs[:, 3].sum()), elems, out, 0)
        dst = torch.zeros(bound, dtype=torch.uint8, device=DEV)
        more = dict(out_dtype=out, summary_mask=0, keep_mask=None if keep is None else torch.from_numpy(keep).to(DEV),
                    row_index=None if idx is None else torch.from_numpy(idx).to(DEV))
        B.observe_into(1, x, reqs, dst, seq=0, step_id=0, stream=s, **more)
        assert np.array_equal(dst.cpu().numpy()[:ref.size], ref), n_rows
        with B.Ring((bound + bound // 2) // 64 * 64, 2 * bound) as ring:
            for seq in range(2):                    # (the second one wraps)
                ring.observe_tensor(1, x, reqs, step_id=0, stream=s, **more)
                ring.drain(B.DRAIN_FLUSH)
                (view,) = ring.poll_host()
                got = view.bytes().copy()
                got[8:16] = 0                       # (its sequence number)
                assert np.array_equal(got, ref), (n_rows, seq)
                ring.release_host(view.seq)


@pytest.mark.parametrize("elems,out", [(512, 1), (568, 2), (640, 4), (517, 4)])
def test_batches(B, elems, out):
    s = torch.cuda.current_stream().cuda_stream
    reqs = np.array([[i, i, 0, 1, 1] for i in range(250)], dtype=np.uint32)
    for n in (47, 50):
        xs = [prng.randn_bf16(p, 250 * elems, DEV).view(250, elems) for p in range(n)]
        size = B.record_bytes(250, 250, elems, out, 0)
        with B.Ring((n + 3) * size, (n + 3) * size) as ring:
            for step in range(2):
                ring.observe_batch(range(n), xs, reqs, step_id=step, stream=s, out_dtype=out, summary_mask=0)
                ring.drain(B.DRAIN_FLUSH)
                views = ring.poll_host(n)
                assert len(views) == n
                for p, v in enumerate(views):
                    ref = orc.build_record(xs[p].cpu(), reqs, seq=step * n + p, step_id=step, point_id=p, out_dtype=out, summary_mask=0)
                    assert np.array_equal(v.bytes(), ref), (n, step, p)
                ring.release_host(views[-1].seq)


@pytest.mark.parametrize("elems,out", [(256, 1), (250, 4)])
@pytest.mark.parametrize("rounds", [5, 9, 10, 20, 21])
def test_ragged_batches(B, elems, out, rounds):
    """Both sides of the lines where a batch's workgroups are given another share of it (1280 items of 1024 units to a round)."""
    s = torch.cuda.current_stream().cuda_stream
    n, units = 8, -(-elems * 2 // 16)
    each = (rounds * 1280 - 60) * 1024 // units // n // 50
    reqs = np.array([[i, each * i, 0, each - (i % 3), 1] for i in range(50)], dtype=np.uint32)
    xs = [prng.randn_bf16(p, 50 * each * elems, DEV).view(-1, elems) for p in range(n)]
    size = B.record_bytes(50, int(reqs[:, 3].sum()), elems, out, 0)
    with B.Ring((n + 1) * size, (n + 1) * size) as ring:
        ring.observe_batch(range(n), xs, reqs, step_id=3, stream=s, out_dtype=out, summary_mask=0)
        ring.drain(B.DRAIN_FLUSH)
        views = ring.poll_host(n)
        assert len(views) == n
        for p in (0, 3, n - 1):
            ref = orc.build_record(xs[p].cpu(), reqs, seq=p, step_id=3, point_id=p, out_dtype=out, summary_mask=0)
            assert np.array_equal(views[p].bytes(), ref), p
        ring.release_host(views[-1].seq)
