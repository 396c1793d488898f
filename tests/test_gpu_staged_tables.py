"""Request tables that are staged by a launch of their own, at the sizes where the number and kind of those launches
changes (896 and 3072 words), called directly and replayed from a graph; and statistics of rows of 256 units, a wavefront
each, by a launch that reads more than the memory-side cache holds (shorter rows: test_gpu_row_routes.py)."""
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


@pytest.mark.parametrize("n", [179, 180, 614, 615, 1024])
@pytest.mark.parametrize("width", [24, 520])
def test_tables(B, n, width):
    x = prng.randn_bf16(n, 1100 * width, DEV).view(1100, width)
    at = np.random.default_rng(n).permutation(1100)[:n]
    reqs = np.array([[7 * i, a, 0, 1, 1] for i, a in enumerate(at)], dtype=np.uint32)
    ref = orc.build_record(x.cpu(), reqs, seq=3, step_id=4, point_id=5, out_dtype=4, summary_mask=0)
    dst = torch.zeros(ref.size, dtype=torch.uint8, device=DEV)
    call = lambda: B.observe_into(5, x, reqs, dst, seq=3, step_id=4, out_dtype=4,      # noqa: E731
                                  stream=torch.cuda.current_stream().cuda_stream)
    call()
    assert np.array_equal(dst.cpu().numpy(), ref)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        dst.zero_()
        torch.cuda.synchronize()
        g.replay()
        assert np.array_equal(dst.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_short_rows_past_the_cache(B, dtype):
    width = 2048 if dtype == torch.bfloat16 else 1024
    rows = 66000
    x = prng.randn_bf16(3, rows * width, DEV).view(rows, width).to(dtype)
    reqs = np.array([[i, 2200 * i, 0, 2200, 1] for i in range(30)], dtype=np.uint32)
    dst = torch.zeros(B.record_bytes(30, rows, width, 0, 7), dtype=torch.uint8, device=DEV)
    B.observe_into(5, x, reqs, dst, seq=0, step_id=0, out_dtype=0, summary_mask=7, stream=torch.cuda.current_stream().cuda_stream)
    some = slice(2200 * 13, 2200 * 15)                                 # (the oracle takes its time)
    ref = orc.build_record(x[some].cpu(), np.array([[13, 0, 0, 2200, 1], [14, 2200, 0, 2200, 1]], dtype=np.uint32), seq=0, step_id=0,
                           point_id=5, out_dtype=0, summary_mask=7)
    got = dst.cpu().numpy()[64 + 512:].view(np.float32).reshape(3, -1)[:, some]
    part = ref.copy()
    pad = (4400 * 4 + 63) // 64 * 16
    for k in range(3):
        part[64 + 64:].view(np.float32)[k * pad:k * pad + 4400] = got[k]
    compare_record(part, ref, mean_abs=x[some].float().abs().mean(1).cpu().numpy())
    d = x.double()
    for k, want in enumerate((d.square().sum(1).sqrt(), d.mean(1), d.abs().amax(1))):
        all_rows = torch.from_numpy(dst.cpu().numpy()[64 + 512:].view(np.float32).reshape(3, -1)[k, :rows].copy()).double().to(DEV)
        assert float((all_rows - want).norm() / want.norm()) < 2e-6
