"""Kernel variants that only certain launches take: statistics of short rows by a launch that reads more than the memory-side cache
holds; replayed steps whose selection grows, with summaries (the row loops of a wavefront and of a workgroup per row); and
selections of several rows per request whose table fits a launch's arguments only without a word per row.  Against the oracle."""
import types

import numpy as np
import pytest
import torch

import oracle as orc
from workloads import prng
from _util import compare_record

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TORCH = {1: torch.bfloat16, 2: torch.float16, 3: torch.float32}


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


def _stream():
    return torch.cuda.current_stream().cuda_stream


# (test_launch_plans holds that these are read past the cache, and not by the kernel for longer rows)
@pytest.mark.parametrize("src,elems,rows", [(1, 1024, 132000), (1, 256, 530000), (2, 1000, 135000), (3, 512, 132000), (1, 2040, 66500)])
def test_short_rows_past_the_cache(B, src, elems, rows):
    x = prng.randn_bf16(elems, rows * elems, DEV).view(rows, elems).to(TORCH[src])
    x[1, 0], x[rows - 2, elems - 1], x[4, 1:9] = float("nan"), float("-inf"), -float("nan")
    n = 40
    each = rows // n
    reqs = np.array([[i, each * i, 0, each - i % 3, 1] for i in range(n)], dtype=np.uint32)
    at = np.concatenate([q[1] + np.arange(q[3]) for q in reqs])
    dst = torch.zeros(B.record_bytes(n, at.size, elems, 0, 7), dtype=torch.uint8, device=DEV)
    B.observe_into(5, x, reqs, dst, seq=3, step_id=4, out_dtype=0, summary_mask=7, stream=_stream())
    ref = orc.build_record(x.cpu(), reqs, seq=3, step_id=4, point_id=5, out_dtype=0, summary_mask=7)
    compare_record(dst.cpu().numpy(), ref, mean_abs=x.float().abs().mean(1).cpu().numpy()[at])


@pytest.mark.parametrize("heads,take,dim,tokens", [(8, 2, 128, 20000), (8, 8, 256, 2400)])
def test_paged_rows_past_the_cache(B, heads, take, dim, tokens):
    """Slices of three caches in one launch."""
    n_seqs, size, layers = 10, 16, 3
    per_seq = tokens // size
    n_blocks = n_seqs * per_seq + 5
    caches = [prng.randn_bf16(layer, n_blocks * size * heads * dim, DEV).view(n_blocks, size, heads, dim) for layer in range(layers)]
    table = torch.from_numpy(np.random.default_rng(1).permutation(n_blocks)[:n_seqs * per_seq].astype(np.int32).reshape(n_seqs, per_seq))
    pick = list(range(heads))[-take:]
    paged = types.SimpleNamespace(block_table=table.to(DEV), block_size=size, n_heads=heads, head_dim=dim, heads_sel=pick)
    reqs = np.array([[i, i, i, tokens - 2 * i, 1] for i in range(n_seqs)], dtype=np.uint32)
    rows = int(reqs[:, 3].sum())
    assert layers * rows * take * dim * 2 > 256 << 20
    size_b = B.record_bytes(n_seqs, rows, take * dim, 0, 5)
    with B.Ring(4 * size_b, 4 * size_b) as ring:
        ring.observe_batch(range(layers), caches, reqs, step_id=1, stream=_stream(), out_dtype=0, summary_mask=5, paged=paged)
        ring.drain(B.DRAIN_FLUSH)
        views = ring.poll_host()
        assert len(views) == layers
        for p, v in enumerate(views):
            # (gathered here: the rows in their order, for the oracle's dense form; table and counts are the same)
            t = torch.cat([torch.arange(int(q[2]), int(q[2] + q[3])) for q in reqs])
            s = torch.from_numpy(np.repeat(reqs[:, 1].astype(np.int64), reqs[:, 3]))
            flat = caches[p].cpu()[table[s, t // size].long(), t % size][:, pick].reshape(rows, take * dim)
            at = np.concatenate([[0], np.cumsum(reqs[:, 3])[:-1]])
            dense = np.array([[q[0], a - q[2], q[2], q[3], 1] for q, a in zip(reqs.astype(np.int64), at)])
            dense[:, 1] %= 2 ** 32
            dense = dense.astype(np.uint32)
            ref = orc.build_record(flat, dense, seq=p, step_id=1, point_id=p, out_dtype=0, summary_mask=5,
                                   row_index=np.arange(rows, dtype=np.int32))
            ref[31] = 1                                             # (flags: paged, not indexed)
            compare_record(v.bytes(), ref, what=f"cache {p}")


@pytest.mark.parametrize("src,elems", [(1, 1536), (1, 4096), (3, 4096), (1, 9000), (1, 2049)])
@pytest.mark.parametrize("out", [0, 1])
def test_replayed_steps_with_summaries_whose_selection_grows(B, src, elems, out):
    rows = 1600
    out = 3 if out and src == 3 else out
    x = prng.randn_bf16(elems, rows * elems, DEV).view(rows, elems).to(TORCH[src])
    scale = x.float().abs().mean(1).cpu().numpy()
    few = np.array([[i, 40 * i, 0, 1 + i % 2, 1] for i in range(6)], dtype=np.uint32)
    grown = np.array([[i, 2 * i, 1, 500 - 90 * i, 3 if i == 0 else 1] for i in range(6)], dtype=np.uint32)
    grown[3, 3] = 0
    s = torch.cuda.Stream()
    with B.Ring(128 << 20, 256 << 20) as ring:
        step = B.Step(ring, 4)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        step.capture_begin()
        with torch.cuda.graph(g, stream=s):
            for p in range(2):
                step.observe_tensor(p, x, few, stream=torch.cuda.current_stream().cuda_stream, out_dtype=out, summary_mask=7)
        step.seal()
        seq = 0
        for k, reqs in enumerate([few, grown, few, grown, grown]):
            step.update(0, reqs)
            with torch.cuda.stream(s):
                step.begin(k, s.cuda_stream)
                g.replay()
                step.end(s.cuda_stream)
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert len(views) == 2
            at = np.concatenate([q[1] + q[2] + q[4] * np.arange(q[3]) for q in reqs.astype(np.int64)])
            for p, v in enumerate(views):
                ref = orc.build_record(x.cpu(), reqs, seq=seq + p, step_id=k, point_id=p, out_dtype=out, summary_mask=7)
                compare_record(v.bytes(), ref, what=f"{k} {p}", mean_abs=scale[at])
            ring.release_host(views[-1].seq)
            seq += 2
        step.destroy()


@pytest.mark.parametrize("elems", [520, 4096])
@pytest.mark.parametrize("mask", [0, 5])
@pytest.mark.parametrize("n,each", [(1, 827), (1, 828), (16, 47), (16, 50), (64, 8), (64, 9), (65, 8), (65, 9)])
def test_tables_on_both_sides_of_a_launchs_arguments(B, elems, mask, n, each):
    """832 words: five per request, and one per row where the decode-shaped kernel takes the launch."""
    x = prng.randn_bf16(n + each, 1100 * elems, DEV).view(1100, elems)
    reqs = np.array([[3 * i, 0, (1100 - each) * i // max(1, n - 1), each, 1] for i in range(n)], dtype=np.uint32)
    for out in (1, 4):
        ref = orc.build_record(x.cpu(), reqs, seq=0, step_id=9, point_id=5, out_dtype=out, summary_mask=mask)
        dst = torch.zeros(ref.size + 64, dtype=torch.uint8, device=DEV)
        B.observe_into(5, x, reqs, dst, seq=0, step_id=9, out_dtype=out, summary_mask=mask, stream=_stream())
        got = dst.cpu().numpy()
        assert not got[ref.size:].any()
        compare_record(got[:ref.size], ref, what="into")
        with B.Ring((2 * ref.size + 4096) // 64 * 64, (2 * ref.size + 4096) // 64 * 64) as ring:
            ring.observe_tensor(5, x, reqs, step_id=9, stream=_stream(), out_dtype=out, summary_mask=mask)
            ring.drain(B.DRAIN_FLUSH)
            (view,) = ring.poll_host()
            assert np.array_equal(view.bytes(), got[:ref.size])     # (bit for bit, the summaries too)
