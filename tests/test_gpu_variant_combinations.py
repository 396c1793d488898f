"""Kernel variants in the launches that their own tests leave out: a wavefront per row in dmi_observe_into;
a wavefront per row and rows off the 16-byte grid in batched nodes of a replayed step, and in batches part of which
is dropped, by the host or by the kernel.  Every record against the oracle (tolerances as in _util)."""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import prng
from _util import compare_record

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("elems,lead,out,mask", [(2056, 0, 0, 7), (2056, 0, 4, 5), (4096, 0, 1, 7), (6144, 0, 0, 5),
                                                 (4093, 0, 1, 5), (2057, 3, 0, 7), (6100, 1, 0, 3)])
@pytest.mark.parametrize("n", [40, 200])        # the request table travels with the launch, or is staged
@pytest.mark.parametrize("how", ["ragged", "keep", "index"])
def test_into_with_a_wavefront_per_row(B, elems, lead, out, mask, n, how):
    per, src = -(-2100 // n), 400
    x = prng.randn_bf16(elems + n, src * (elems + lead), DEV).view(src, elems + lead)[:, lead:]
    rng = np.random.default_rng(elems + n)
    counts = np.full(n, per)
    counts[1::9] = 0
    counts[2::9] += per                         # (what the requests without rows leave out)
    assert counts.sum() >= 2048
    reqs = np.array([[i, int(rng.integers(0, src - 2 * per)), 0, c, 1] for i, c in enumerate(counts)], dtype=np.uint32)
    keep = (rng.integers(0, 4, n) > 0).astype(np.uint8) if how == "keep" else None
    index = rng.integers(0, src, counts.sum()).astype(np.int32) if how == "index" else None
    s = torch.cuda.current_stream()
    bound = B.record_bytes(n, int(counts.sum()), elems, out, mask)
    dst = torch.full((bound + 64,), 0xC3, dtype=torch.uint8, device=DEV)
    size = B.observe_into(4, x, reqs, dst[:bound], seq=3, step_id=8, out_dtype=out, summary_mask=mask, stream=s.cuda_stream,
                          keep_mask=None if keep is None else torch.from_numpy(keep).to(DEV),
                          row_index=None if index is None else torch.from_numpy(index).to(DEV))
    assert size == bound
    ref = orc.build_record(x.cpu(), reqs, seq=3, step_id=8, point_id=4, out_dtype=out, summary_mask=mask, keep_mask=keep,
                           row_index=index)
    got = dst.cpu().numpy()
    rows = index if index is not None else np.concatenate([q[1] + np.arange(q[3]) for q in reqs])
    kept = np.ones(rows.size, bool) if keep is None else np.repeat(keep, counts).astype(bool)
    compare_record(got[:ref.size], ref, mean_abs=x.float().abs().mean(1).cpu().numpy()[rows[kept]])
    assert np.all(got[ref.size:] == 0xC3)


VARIANTS = {                # elements, out, summaries of 4 x 600 rows
    "wave": (4096, 0, 7),
    "wave_with_rows": (3072, 1, 5),
    "wave_loose": (4093, 1, 7),
    "loose": (1001, 1, 0),
    "loose_short": (1001, 4, 5),
    "loose_rows": (4101, 1, 5),
}
N, ROWS = 4, 600


def _requests(ragged):
    if not ragged:
        return np.array([[i, ROWS - 1 - i, 0, 1, 1] for i in range(ROWS)], dtype=np.uint32)
    counts = [0, 1, 299, 0, 300]
    return np.array([[i, 0, 0, c, 1] for i, c in enumerate(counts)], dtype=np.uint32)


def _check(v, x, reqs, *, step, point, out, mask, keep=None):
    rows = np.concatenate([q[1] + q[2] + np.arange(q[3]) * q[4] for q in reqs]).astype(np.int64)
    if keep is not None:
        rows = rows[np.repeat(keep, reqs[:, 3]).astype(bool)]
    ref = orc.build_record(x.cpu(), reqs, seq=v.seq, step_id=step, point_id=point, out_dtype=out, summary_mask=mask, keep_mask=keep)
    compare_record(v.bytes(), ref, what=f"seq {v.seq}", mean_abs=x.float().abs().mean(1).cpu().numpy()[rows])


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("ragged", [False, True])
def test_batched_node_of_a_replayed_step(B, variant, ragged):
    """Three replays with room for everything, then two under best effort with room for two and a half of the
    four records: the launch was captured before either was known."""
    elems, out, mask = VARIANTS[variant]
    reqs = _requests(ragged)
    rb = B.record_bytes(len(reqs), ROWS, elems, out, mask)
    xs = [torch.empty(ROWS, elems, dtype=torch.bfloat16, device=DEV) for _ in range(N)]
    s = torch.cuda.current_stream()
    points = [5, 6, 7, 8]
    for mode, cap, fits in ((B.POLICY_BLOCK, 5 * rb, 4), (B.POLICY_DROP_NEWEST, 2 * rb + rb // 2 // 64 * 64, 2)):
        with B.Ring(cap, 8 * rb, max_reqs_per_observe=1024) as ring:
            ring.debug_fill_rings(0xA5)
            ring.set_policy(mode)
            step = B.Step(ring, N)
            graph = torch.cuda.CUDAGraph()
            step.capture_begin()
            with torch.cuda.graph(graph):
                step.observe_batch(points, xs, reqs, stream=torch.cuda.current_stream().cuda_stream, out_dtype=out, summary_mask=mask)
            step.seal()
            for r in range(3 if mode == B.POLICY_BLOCK else 2):
                for p, x in enumerate(xs):
                    x.copy_(prng.randn_bf16(100 * r + p, ROWS * elems, DEV).view(ROWS, elems))
                assert step.begin(r, s.cuda_stream) == B.OK
                graph.replay()
                step.end(s.cuda_stream)
                ring.drain(B.DRAIN_FLUSH)
                views = ring.poll_host()
                assert [v.seq for v in views] == [N * r + i for i in range(fits)]
                for i, v in enumerate(views):
                    _check(v, xs[i], reqs, step=r, point=points[i], out=out, mask=mask)
                ring.release_host(views[-1].seq)
            torch.cuda.synchronize()
            step.destroy()


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("keep", [False, True])     # a caller's keep vector: what fits is known to the kernel alone
def test_batch_that_drops_part_of_itself(B, variant, ragged, keep):
    elems, out, mask = VARIANTS[variant]
    reqs = _requests(ragged)
    kv = np.ones(len(reqs), dtype=np.uint8)
    if keep:
        kv[2::5] = 0
    rows = int(reqs[:, 3][kv == 1].sum())
    rb = B.record_bytes(len(reqs), rows, elems, out, mask)
    bound = B.record_bytes(len(reqs), ROWS, elems, out, mask)
    cap = max(2 * rb + rb // 2, bound) // 64 * 64
    fits = cap // rb
    assert 1 <= fits < N
    xs = [prng.randn_bf16(p, ROWS * elems, DEV).view(ROWS, elems) for p in range(N)]
    s = torch.cuda.current_stream()
    with B.Ring(cap, 8 * bound, max_reqs_per_observe=1024) as ring:
        ring.debug_fill_rings(0xA5)
        ring.set_policy(B.POLICY_DROP_NEWEST)
        km = torch.from_numpy(kv).to(DEV) if keep else None
        for step in range(3):
            ring.observe_batch([1, 2, 3, 4], xs, reqs, step_id=step, stream=s.cuda_stream, out_dtype=out, summary_mask=mask, keep_mask=km)
            s.synchronize()
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert [v.seq for v in views] == [N * step + i for i in range(fits)]
            for i, v in enumerate(views):
                _check(v, xs[i], reqs, step=step, point=i + 1, out=out, mask=mask, keep=kv if keep else None)
            ring.release_host(views[-1].seq)
        st = ring.get_stats()
        assert (st.captured_records, st.dropped_records) == (3 * fits, 3 * (N - fits))
        assert st.dropped_bytes == 3 * (N - fits) * rb and st.dropped_rows == 3 * (N - fits) * rows
        assert [ring.get_point_drops(p) for p in (1, 2, 3, 4)] == [0 if i < fits else 3 for i in range(N)]
