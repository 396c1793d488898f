"""dmi_observe_into: request tables that travel with the launch (at most 832 words: 5 per request, and the source
row of every listed row where a small selection lists several rows per request) and longer ones that are
staged, on both sides of the line, in both kernels, back to back and inside a graph: the records
are dmi_observe's byte for byte."""
import numpy as np
import pytest
import torch

from workloads import prng

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available()
    from paper_2605_11093_amd import binding
    binding.lib()
    return binding


def _both(B, x, reqs, *, out_dtype=1, summary_mask=0, keep=None, index=None):
    s = torch.cuda.current_stream()
    reqs = np.asarray(reqs, dtype=np.uint32).reshape(-1, 5)
    km = None if keep is None else torch.from_numpy(np.asarray(keep, dtype=np.uint8)).to(DEV)
    ri = None if index is None else torch.from_numpy(np.asarray(index, dtype=np.int32)).to(DEV)
    out = torch.full((16 << 20,), 0xC3, dtype=torch.uint8, device=DEV)
    n = B.observe_into(2, x, reqs, out, seq=0, step_id=9, out_dtype=out_dtype, summary_mask=summary_mask, keep_mask=km,
                       row_index=ri, stream=s.cuda_stream)
    with B.Ring(16 << 20, 16 << 20, max_reqs_per_observe=1024) as ring:
        ring.observe_tensor(2, x, reqs, step_id=9, stream=s.cuda_stream, out_dtype=out_dtype, summary_mask=summary_mask,
                            keep_mask=km, row_index=ri)
        ring.drain(B.DRAIN_FLUSH)
        (v,) = ring.poll_host()
        want = v.bytes()
    host = out.cpu().numpy()
    assert want.size <= n and np.array_equal(host[:want.size], want)
    assert np.all(host[want.size:] == 0xC3)


@pytest.mark.parametrize("n", [1, 2, 165, 166, 167, 256, 1024])
@pytest.mark.parametrize("how", ["in_order", "slots", "index", "keep", "fp32"])
def test_one_row_per_request(B, n, how):
    x = prng.randn_bf16(n, 1024 * 512, DEV).view(1024, 512)
    rng = np.random.default_rng(n)
    at = np.arange(n) if how == "in_order" else rng.permutation(1024)[:n]
    reqs = [[100 + i, int(at[i]), 0, 1, 1] for i in range(n)]
    if how == "fp32":
        _both(B, x.float(), reqs, out_dtype=3, summary_mask=5)
    else:
        _both(B, x, reqs, summary_mask=5, index=at[::-1].copy() if how == "index" else None,
              keep=rng.integers(0, 2, n) if how == "keep" else None)


@pytest.mark.parametrize("n,rows", [(1, 827), (1, 828), (32, 21), (40, 16), (150, 2), (166, 7), (167, 7)])
@pytest.mark.parametrize("keep", [False, True])
def test_several_rows_per_request(B, n, rows, keep):
    x = prng.randn_bf16(n, 1400 * 256, DEV).view(1400, 256)
    reqs = [[i, i * rows, 0, rows if i % 5 else rows // 2, 1] for i in range(n)]
    _both(B, x, reqs, out_dtype=4, keep=[i % 3 != 1 for i in range(n)] if keep else None)
    _both(B, x[:, 3:], reqs, out_dtype=2, summary_mask=2, keep=[1] * n if keep else None)


def test_back_to_back_calls_keep_their_tables_and_a_graph_replays_them(B):
    x = prng.randn_bf16(4, 64 * 256, DEV).view(64, 256)
    s = torch.cuda.current_stream()
    sets = [np.array([[1000 * k + i, (i * 7 + k) % 64, 0, 1, 1] for i in range(60)], dtype=np.uint32) for k in range(6)]
    outs = [torch.zeros(64 << 10, dtype=torch.uint8, device=DEV) for _ in sets]
    def want(k):
        return x[torch.from_numpy(sets[k][:, 1].astype(np.int64)).to(DEV)].contiguous().view(torch.uint8).reshape(-1)
    def check():
        for k, o in enumerate(outs):
            at = 64 + 960
            assert torch.equal(o[at:at + 60 * 512], want(k)), k
            assert o[64:64 + 960].cpu().numpy().view(np.uint32).reshape(60, 4)[:, 0].tolist() == sets[k][:, 0].tolist()
    for k, o in enumerate(outs):
        B.observe_into(1, x, sets[k], o, seq=k, step_id=0, stream=s.cuda_stream)
    check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h = torch.cuda.current_stream().cuda_stream
        for k, o in enumerate(outs):
            B.observe_into(1, x, sets[k], o, seq=k, step_id=0, stream=h)
    for r in range(4):
        x.copy_(prng.randn_bf16(50 + r, 64 * 256, DEV).view(64, 256))
        for o in outs:
            o.zero_()
        g.replay()
        torch.cuda.synchronize()
        check()
