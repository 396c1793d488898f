"""A flush that copies what the launches' notes say is complete while later captures run: every kernel that leaves notes, in
replayed steps and in single calls, with inputs that change between the flushes, against the oracle's records; and with work in
front of the last capture that takes longer than the copies, so that some must have been made by notes."""
import numpy as np
import pytest
import torch

import oracle as orc
from workloads import prng

from _util import compare_record

pytestmark = pytest.mark.gpu

CASES = [       # records, rows of each, width, source, stored as, rings
    (20, 64, 4096, "bf16", "bf16", 12 << 20),       # the decode-shaped kernel; the ring wraps in every other flush
    (8, 64, 16384, "fp32", "fp32", 64 << 20),       # capture_rows_kernel
    (16, 2048, 128, "bf16", "bf16", 64 << 20),      # the general kernel, rows dealt flat
    (3, 64, 4096, "bf16", "fp8", 64 << 20),         # less than a copy is worth in front of the last note
]


@pytest.mark.parametrize("how", ["replay", "calls"])
@pytest.mark.parametrize("n,rows,width,dtype,out,ring_bytes", CASES)
def test_every_flush_delivers_the_oracles_records(how, n, rows, width, dtype, out, ring_bytes):
    from paper_2605_11093_amd import binding as B
    from paper_2605_11093_amd import hookpoint as H
    code = {"bf16": B.DT_BF16, "fp32": B.DT_FP32, "fp8": B.DT_FP8}
    x = [torch.empty(rows, width, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda:0") for _ in range(n)]
    reqs = np.array([[50 + i, i, 0, 1, 1] for i in range(rows)], dtype=np.uint32)
    s = torch.cuda.current_stream().cuda_stream
    with B.Ring(ring_bytes, ring_bytes, max_reqs_per_observe=rows, block_timeout_ms=5000) as ring:
        if how == "replay":
            ctx = H.StepContext()
            hooks = [H.HookPoint(ring, p, ctx, out_dtype=code[out]) for p in range(n)]
            graph = torch.cuda.CUDAGraph()
            with ctx.capture(ring, reqs, max_observes=n):
                with torch.cuda.graph(graph):
                    for hook, t in zip(hooks, x):
                        hook(t)
        seq = 0
        for flush in range(4):
            for i, t in enumerate(x):
                t.copy_(prng.randn_bf16(1000 * flush + i, rows * width, "cuda:0").view(rows, width))
            if how == "replay":
                ctx.begin_replay(flush, s)
                graph.replay()
                ctx.end_replay(s)
            else:
                for p, t in enumerate(x):
                    ring.observe_tensor(p, t, reqs, step_id=flush, out_dtype=code[out], stream=s)
            ring.drain(B.DRAIN_FLUSH)
            views = ring.poll_host()
            assert [v.seq for v in views] == list(range(seq, seq + n))
            for p in sorted({0, 1, n // 2, n - 2, n - 1}):
                ref = orc.build_record(x[p].cpu(), reqs, seq=seq + p, step_id=flush, point_id=p, out_dtype=code[out])
                compare_record(views[p].bytes(), ref)
            whole = [np.frombuffer(v.bytes(), dtype=np.uint8) for v in views]
            if out == dtype:                # the others' payload as a plain copy of their source
                head = 64 + -(-16 * rows // 64) * 64
                for p, t in enumerate(x):
                    want = t.view(torch.uint8).cpu().numpy().reshape(-1)
                    assert np.array_equal(whole[p][head:head + want.size], want), (flush, p)
            ring.release_host(views[-1].seq)
            seq += n
        st = ring.get_stats()
        assert st.captured_records == seq and st.drained_bytes == st.captured_bytes == st.released_bytes
        assert st.dev_ring_high_water <= ring_bytes and st.host_ring_high_water <= ring_bytes


@pytest.mark.parametrize("how", ["replay", "calls"])
@pytest.mark.parametrize("rows,width,dtype", [(128, 4096, "bf16"), (64, 16384, "fp32"), (4096, 128, "bf16")])
def test_a_flush_copies_by_notes_while_the_last_capture_waits(how, rows, width, dtype):
    """Of five records of 1 to 4 MB four are captured at once, of which the notes tell of three; the fifth's capture waits behind
    some 2 ms of matrix products.  Two copies or more mean that notes were followed: no event lies between the captures."""
    from paper_2605_11093_amd import binding as B
    from paper_2605_11093_amd import hookpoint as H
    torch_type = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = [prng.randn_bf16(60 + i, rows * width, "cuda:0").view(rows, width).to(torch_type) for i in range(5)]
    reqs = np.array([[50 + i, i, 0, 1, 1] for i in range(rows)], dtype=np.uint32)
    m = prng.randn_bf16(3, 8192 * 8192, "cuda:0").view(8192, 8192)
    product = torch.empty_like(m)
    s = torch.cuda.current_stream().cuda_stream

    def work():
        for _ in range(3):
            torch.mm(m, m, out=product)

    work()
    with B.Ring(64 << 20, 64 << 20, max_reqs_per_observe=rows, block_timeout_ms=5000) as ring:
        if how == "replay":
            ctx = H.StepContext()
            hooks = [H.HookPoint(ring, p, ctx) for p in range(5)]
            graph = torch.cuda.CUDAGraph()
            with ctx.capture(ring, reqs, max_observes=5):
                with torch.cuda.graph(graph):
                    for p, hook in enumerate(hooks):
                        if p == 4:
                            work()
                        hook(x[p])
        for flush in range(3):
            torch.cuda.synchronize()
            before = ring.get_stats().drain_batches
            if how == "replay":
                ctx.begin_replay(flush, s)
                graph.replay()
                ctx.end_replay(s)
            else:
                for p, t in enumerate(x):
                    if p == 4:
                        work()
                    ring.observe_tensor(p, t, reqs, step_id=flush, stream=s)
            ring.drain(B.DRAIN_FLUSH)
            assert ring.get_stats().drain_batches - before >= 2
            views = ring.poll_host()
            assert [v.seq for v in views] == list(range(5 * flush, 5 * flush + 5))
            for p in (0, 3, 4):
                ref = orc.build_record(x[p].cpu(), reqs, seq=5 * flush + p, step_id=flush, point_id=p,
                                       out_dtype=B.DT_BF16 if dtype == "bf16" else B.DT_FP32)
                compare_record(views[p].bytes(), ref)
            ring.release_host(views[-1].seq)
