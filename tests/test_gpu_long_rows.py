"""Rows that a launch finds by itself (dense, one row per request or up to 64 ragged requests): those of 64 units and more
stored without summaries, a wavefront per 256 units, and those of more than 128 units with them, a wavefront or a
workgroup per row: row lengths at the edges of a
step (one unit, a part and a unit, odd numbers of units), rows off the 16-byte grid, requests without rows, keep
vectors, bad indexes, one row per request in and out of order, 64 requests and 65 (the general kernel again),
records that wrap at the end of the ring, NaN and infinities; singly, batched, partly dropped, into the caller's
memory, and in replayed steps whose selection grows.  Byte for byte against the oracle (summaries: _util's tolerances)."""
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


def _source(rows, elems, lead, src, seed=1):
    x = prng.randn_bf16(seed + elems, rows * (elems + lead), DEV).view(rows, elems + lead)[:, lead:].to(TORCH[src])
    x[1, 0], x[2, elems - 1], x[3, elems // 2] = float("nan"), float("-inf"), float("inf")
    x[4, 1:9] = -float("nan")
    return x


def _reqs(n, per, rows, one=False, shuffled=False):
    """n requests: of one row each, or ragged ones, every fifth without rows, every third with a stride"""
    rng = np.random.default_rng(n + per)
    if one:
        at = rng.permutation(rows)[:n] if shuffled else np.arange(n) + 2
        return np.array([[i, a, 0, 1, 1] for i, a in enumerate(at)], dtype=np.uint32)
    out = []
    for i in range(n):
        c = 0 if i % 5 == 4 else int(rng.integers(1, 2 * per))
        step = 3 if i % 3 == 0 else 1
        out.append([100 + i, int(rng.integers(0, rows - c * step)), 0, c, step])
    return np.array(out, dtype=np.uint32)


def _selections(rows):
    rng = np.random.default_rng(9)
    few, many, more = _reqs(7, 30, rows), _reqs(64, 8, rows), _reqs(65, 8, rows)
    index = rng.integers(0, rows, int(few[:, 3].sum())).astype(np.int32)
    index[::17], index[5] = rows, -1
    keep = np.array([1, 0, 1, 1, 1, 0, 1], dtype=np.uint8)
    return {"ragged": (few, None, None), "64": (many, None, None), "65": (more, None, None), "keep": (few, keep, None),
            "none kept": (few, np.zeros(7, dtype=np.uint8), None), "index": (few, None, index),
            "index keep": (few, keep, index), "one": (_reqs(1100, 1, rows, True), None, None),
            "slots": (_reqs(1100, 1, rows, True, True), None, None), "no requests": (few[:0], None, None)}


@pytest.mark.parametrize("elems,lead", [(512, 0), (520, 0), (2040, 0), (2048, 0), (2056, 0), (4096, 0), (14336, 0), (505, 0), (2041, 0),
                                        (2049, 3), (4099, 1), (2063, 0)])
@pytest.mark.parametrize("src,out", [(1, 1), (1, 2), (1, 4), (3, 3)])
def test_records_against_the_oracle(B, elems, lead, src, out):
    if src == 3:
        elems //= 2
    rows = 1300
    x = _source(rows, elems, lead, src)
    xc = x.cpu()
    s = torch.cuda.current_stream().cuda_stream
    # (a ring of two and a bit of the largest records: they wrap at every alignment of the 64-byte grid)
    sel = _selections(rows)
    biggest = max(B.record_bytes(len(q), int(q[:, 3].sum()), elems, out, 0) for q, _, _ in sel.values())
    with B.Ring(biggest * 2 + 4096 + 64 * 5, biggest * 3, max_reqs_per_observe=2048) as ring:
        ring.debug_fill_rings(0xA5)
        bad = 0
        for k, (name, (reqs, keep, index)) in enumerate(sel.items()):
            ring.observe_tensor(3, x, reqs, step_id=k, stream=s, out_dtype=out, summary_mask=0,
                                keep_mask=None if keep is None else torch.from_numpy(keep).to(DEV),
                                row_index=None if index is None else torch.from_numpy(index).to(DEV))
            ring.drain(B.DRAIN_FLUSH)
            (view,) = ring.poll_host()
            y = torch.cat([xc, torch.zeros(1, elems, dtype=xc.dtype)])
            idx = None if index is None else np.where((index < 0) | (index >= rows), rows, index).astype(np.int32)
            ref = orc.build_record(y, reqs, seq=k, step_id=k, point_id=3, out_dtype=out, summary_mask=0, keep_mask=keep,
                                   row_index=idx)
            got = view.bytes()
            assert got.size == ref.size and np.array_equal(got, ref), (name, elems, np.flatnonzero(got != ref)[:8])
            if index is not None:
                kept = np.ones(index.size, bool) if keep is None else np.repeat(keep, reqs[:, 3]).astype(bool)
                bad += int(((idx == rows) & kept).sum())
            ring.release_host(view.seq)
        assert ring.get_stats().bad_rows == bad
        # into the caller's memory: the same records
        for name, (reqs, keep, index) in sel.items():
            if len(reqs) > 1024:
                continue
            bound = B.record_bytes(len(reqs), int(reqs[:, 3].sum()), elems, out, 0)
            dst = torch.full((bound + 64,), 0xC3, dtype=torch.uint8, device=DEV)
            B.observe_into(3, x, reqs, dst[:bound], seq=2, step_id=1, out_dtype=out, stream=s,
                           keep_mask=None if keep is None else torch.from_numpy(keep).to(DEV),
                           row_index=None if index is None else torch.from_numpy(index).to(DEV))
            idx = None if index is None else np.where((index < 0) | (index >= rows), rows, index).astype(np.int32)
            ref = orc.build_record(y, reqs, seq=2, step_id=1, point_id=3, out_dtype=out, summary_mask=0, keep_mask=keep,
                                   row_index=idx)
            got = dst.cpu().numpy()
            assert np.array_equal(got[:ref.size], ref) and np.all(got[bound:] == 0xC3), (name, elems)


@pytest.mark.parametrize("elems,lead", [(1040, 0), (2048, 0), (2047, 0), (1101, 3), (2056, 0), (5120, 0), (5128, 0), (8192, 0), (8200, 0), (16400, 0), (2057, 1), (5125, 0), (8191, 3), (20001, 0)])
@pytest.mark.parametrize("src,out,mask", [(1, 0, 7), (1, 1, 5), (1, 4, 2), (2, 0, 3), (3, 3, 7)])
@pytest.mark.parametrize("many", [False, True])     # rows enough for a wavefront each, or not
def test_summaries_against_the_oracle(B, elems, lead, src, out, mask, many):
    if src == 3:
        elems //= 2
    rows = 260
    x = _source(rows, elems, lead, src)
    xc = torch.cat([x.cpu(), torch.zeros(1, elems, dtype=TORCH[src])])
    scale = np.nan_to_num(xc.float().abs().mean(1).numpy(), posinf=0.0)
    rng = np.random.default_rng(elems)
    counts = [0, 1, 40, 0, 63, 30, 0] if not many else [0, 1, 230, 1400, 0, 500, 36]
    ragged = np.array([[i, int(rng.integers(0, rows - min(c, 250) - 1)), 0, c, 1] for i, c in enumerate(counts)], dtype=np.uint32)
    index = rng.integers(0, rows, sum(counts)).astype(np.int32)
    index[::29] = rows
    keep = np.array([1, 1, 0, 1, 1, 1, 0], dtype=np.uint8)
    spread = np.array([[i, i % rows, 0, 1, 1] for i in range(1200 if not many else 2300)], dtype=np.uint32)
    lots = np.array([[i, (i * 3) % 200, 0, 2 if not many else 33, 1] for i in range(70)], dtype=np.uint32)
    cases = [(ragged, None, index), (ragged, keep, index), (spread, None, None), (lots, None, None), (lots[:64], None, None)]
    s = torch.cuda.current_stream().cuda_stream
    for reqs, k, idx in cases:
        at = idx if idx is not None else np.concatenate([q[1] + np.arange(q[3]) for q in reqs])
        kept = np.ones(at.size, bool) if k is None else np.repeat(k, reqs[:, 3]).astype(bool)
        size = B.record_bytes(len(reqs), at.size, elems, out, mask)
        with B.Ring(2 * size + 4096, 2 * size + 4096, max_reqs_per_observe=4096) as ring:
            for seq in range(2):        # (the second one wraps)
                ring.observe_tensor(2, x, reqs, step_id=seq, stream=s, out_dtype=out, summary_mask=mask,
                                    keep_mask=None if k is None else torch.from_numpy(k).to(DEV),
                                    row_index=None if idx is None else torch.from_numpy(idx).to(DEV))
                ring.drain(B.DRAIN_FLUSH)
                (view,) = ring.poll_host()
                ref = orc.build_record(xc, reqs, seq=seq, step_id=seq, point_id=2, out_dtype=out, summary_mask=mask, keep_mask=k,
                                       row_index=idx)
                compare_record(view.bytes(), ref, what=f"{elems} {len(reqs)}", mean_abs=scale[at[kept]])
                ring.release_host(view.seq)
            assert ring.get_stats().bad_rows == (0 if idx is None else 2 * int(((idx == rows) & kept).sum()))


@pytest.mark.parametrize("elems,lead,shape", [(4096, 0, "one"), (2056, 0, "slots"), (4096, 0, "ragged"), (4099, 0, "ragged")])
def test_batches_that_drop_part_of_themselves(B, elems, lead, shape):
    """Best effort with room for some records of a batch: those that fit are the oracle's, the others are counted."""
    rows, n = 1300, 9
    xs = [_source(rows, elems, lead, 1, seed=p) for p in range(n)]
    reqs = _selections(rows)[shape][0]
    size = B.record_bytes(len(reqs), int(reqs[:, 3].sum()), elems, 4, 0)
    s = torch.cuda.current_stream().cuda_stream
    with B.Ring(5 * size + 128, 16 * size, max_reqs_per_observe=2048) as ring:
        ring.set_policy(B.POLICY_DROP_NEWEST)
        seq = 0
        for step in range(3):
            ring.observe_batch(range(n), xs, reqs, step_id=step, stream=s, out_dtype=4, summary_mask=0)
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert len(views) == 5
            for p, v in enumerate(views):
                ref = orc.build_record(xs[p].cpu(), reqs, seq=seq + p, step_id=step, point_id=p, out_dtype=4, summary_mask=0)
                assert np.array_equal(v.bytes(), ref), (step, p)
            ring.release_host(views[-1].seq)
            seq += n
        assert ring.get_stats().dropped_records == 3 * (n - 5)
        assert [ring.get_point_drops(p) for p in range(n)] == [0] * 5 + [3] * (n - 5)


def test_launches_that_read_more_than_the_cache_holds(B):
    """A launch of more than 256 million bytes takes another load instruction: same bytes."""
    rows, elems = 20000, 8192
    x = prng.randn_bf16(5, rows * elems, DEV).view(rows, elems)
    reqs = np.array([[1, 0, 0, 9000, 1], [2, 9000, 0, 11000, 1]], dtype=np.uint32)
    bound = B.record_bytes(2, rows, elems, 4, 0)
    dst = torch.zeros(bound, dtype=torch.uint8, device=DEV)
    B.observe_into(0, x, reqs, dst, seq=0, step_id=0, out_dtype=4, stream=torch.cuda.current_stream().cuda_stream)
    want = x.float().clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    assert torch.equal(dst[128:128 + rows * elems].view(rows, elems), want)


@pytest.mark.parametrize("elems", [4096, 2049])
def test_replayed_steps_whose_selection_grows(B, elems):
    rows = 1300
    x = _source(rows, elems, 0, 1)
    few = np.array([[i, 40 * i, 0, 3 + i, 1] for i in range(6)], dtype=np.uint32)
    grown = np.array([[i, 2 * i, 1, 400 - 50 * i, 3 if i == 0 else 1] for i in range(6)], dtype=np.uint32)
    s = torch.cuda.Stream()
    with B.Ring(64 << 20, 128 << 20) as ring:
        step = B.Step(ring, 4)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        step.capture_begin()
        with torch.cuda.graph(g, stream=s):
            for p in range(3):
                step.observe_tensor(p, x, few, stream=torch.cuda.current_stream().cuda_stream, out_dtype=4, summary_mask=0)
        step.seal()
        seq = 0
        for k, reqs in enumerate([few, grown, few, grown]):
            step.update(0, reqs)
            with torch.cuda.stream(s):
                step.begin(k, s.cuda_stream)
                g.replay()
                step.end(s.cuda_stream)
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert len(views) == 3
            for p, v in enumerate(views):
                ref = orc.build_record(x.cpu(), reqs, seq=seq + p, step_id=k, point_id=p, out_dtype=4, summary_mask=0)
                assert np.array_equal(v.bytes(), ref), (k, p)
            ring.release_host(views[-1].seq)
            seq += 3
        step.destroy()
