"""Best effort where the kernel itself decides what is dropped (the host does not know the caller's keep vector): rows are
asked for before the head is known, and of a dropped record nothing may arrive, be counted as captured or as a bad row."""
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


@pytest.mark.parametrize("elems,out,mask", [(4096, 4, 0), (520, 1, 0), (4099, 1, 0), (2048, 0, 7), (4096, 1, 5), (9000, 0, 5)])
@pytest.mark.parametrize("indexed", [False, True])
def test_the_kernel_decides(B, elems, out, mask, indexed):
    rows, n, fit = 600, 7, 3
    xs = [prng.randn_bf16(50 + p, rows * elems, DEV).view(rows, elems) for p in range(n)]
    reqs = np.array([[i, 50 * i, 3, 20 + i, 2] for i in range(10)], dtype=np.uint32)
    keep = np.array([1, 0, 1, 1, 0, 1, 1, 1, 0, 1], dtype=np.uint8)
    total, kept = int(reqs[:, 3].sum()), int(reqs[keep > 0, 3].sum())
    at = np.concatenate([q[1] + q[2] + q[4] * np.arange(q[3]) for q in reqs]).astype(np.int32)
    bad = 0
    if indexed:
        at = at[::-1].copy()
        at[[0, 30, total - 1]] = -1, rows, rows + 7
        bad = int((((at < 0) | (at >= rows)) & np.repeat(keep > 0, reqs[:, 3])).sum())
        assert bad
    good = np.where((at < 0) | (at >= rows), rows, at).astype(np.int32)          # (for the oracle: a row of zeros behind the others)
    padded = [torch.cat([x.cpu(), torch.zeros(1, elems, dtype=x.dtype)]) for x in xs]
    size = B.record_bytes(10, kept, elems, out, mask)
    scale = [np.concatenate([x.float().abs().mean(1).cpu().numpy(), [0.0]])[good[np.repeat(keep > 0, reqs[:, 3])]] for x in xs]
    s = torch.cuda.current_stream().cuda_stream
    room = max(fit * size + 64, B.record_bytes(10, total, elems, out, mask))
    room = (room + 63) // 64 * 64
    fit = room // size
    assert 0 < fit < n
    with B.Ring(room, 16 * size + 4096) as ring:
        ring.set_policy(B.POLICY_DROP_NEWEST)
        k = torch.from_numpy(keep).to(DEV)
        idx = torch.from_numpy(at).to(DEV) if indexed else None
        seq = 0
        for step in range(3):
            ring.observe_batch(range(n), xs, reqs, step_id=step, stream=s, out_dtype=out, summary_mask=mask, keep_mask=k, row_index=idx)
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert [v.seq for v in views] == list(range(seq, seq + fit))
            for p, v in enumerate(views):
                ref = orc.build_record(padded[p], reqs, seq=seq + p, step_id=step, point_id=p, out_dtype=out, summary_mask=mask,
                                       keep_mask=keep, row_index=good if indexed else None)
                compare_record(v.bytes(), ref, what=f"{step} {p}", mean_abs=scale[p])
            ring.release_host(views[-1].seq)
            seq += n
        st = ring.get_stats()
        assert (st.captured_records, st.dropped_records, st.bad_rows) == (3 * fit, 3 * (n - fit), 3 * fit * bad)
        assert [ring.get_point_drops(p) for p in range(n)] == [0] * fit + [3] * (n - fit)
