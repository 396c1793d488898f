"""A flush without a drain thread moves small spans with the drain kernel on the producer's own stream.

On the CPU: the host runtime with its threads under ThreadSanitizer and AddressSanitizer (as in
test_host_runtime_sanitizers.py, with a driver of its own).  On the GPU: spans on both sides of the
6 MiB line, rings that wrap inside a span, a host ring without room for all of it, several flushes in a row."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle as orc
from workloads import prng

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CPU = os.path.join(ROOT, "tests", "cpu_runtime")
CSRC = os.path.join(ROOT, "paper_2605_11093_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("sanitizer", ["thread", "address"])
def test_flushes_beside_producer_and_consumer_are_clean_under(tmp_path, sanitizer):
    exe = str(tmp_path / "flush")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", f"-fsanitize={sanitizer}", "-pthread",
           "-I", CPU, "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", exe]
    for src in [os.path.join(CSRC, f) for f in ("dmi_host.hip", "dmi_step.hip", "dmi_exporter.hip")] + \
            [os.path.join(CPU, f) for f in ("fake_hip.cpp", "cpu_kernels.cpp", "flush_driver.cpp")]:
        cmd += ["-x", "c++", src]
    subprocess.check_call(cmd)
    p = subprocess.run([exe, "600"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=280,
                       env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1 exitcode=66", ASAN_OPTIONS="exitcode=67"))
    out = p.stdout.decode(errors="replace")
    assert p.returncode == 0 and "all scenarios passed" in out, out[-6000:]


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1, 2], ids=["default", "copy_engine", "drain_kernel"])
@pytest.mark.parametrize("rows,width,per_flush,dev,host", [
    (4, 256, 1, 1 << 20, 1 << 20),          # a few KB
    (4, 256, 3, 9 * 2176 + 64, 7 * 2176),   # both rings wrap inside a flush
    (64, 4096, 11, 32 << 20, 32 << 20),     # just below 6 MiB
    (64, 4096, 12, 32 << 20, 32 << 20),     # just above
    (64, 4096, 5, 4 << 20, 2 << 20),        # the host ring fills up in the middle
])
def test_flushed_records_are_the_oracles(flags, rows, width, per_flush, dev, host):
    from paper_2605_11093_amd import binding as B
    from _util import compare_record
    x = prng.randn_bf16(9, rows * width, "cuda:0").view(rows, width)
    reqs = np.array([[50 + i, i, 0, 1, 1] for i in range(rows)], dtype=np.uint32)
    size = B.record_bytes(rows, rows, width, B.DT_BF16, 0)
    s, seq, moved = torch.cuda.current_stream().cuda_stream, 0, 0
    with B.Ring(dev, host, flags=flags, block_timeout_ms=200) as ring:
        for flush in range(4):
            for _ in range(per_flush):
                ring.observe_tensor(3, x, reqs, step_id=flush, stream=s)
            want = per_flush
            while want:
                moved += ring.drain(B.DRAIN_FLUSH, allow=(B.ERR_AGAIN,))
                views = ring.poll_host()
                assert views or ring.last_drain_status == B.ERR_AGAIN
                for v in views:
                    assert v.seq == seq
                    ref = orc.build_record(x.cpu(), reqs, seq=seq, step_id=flush, point_id=3, out_dtype=B.DT_BF16)
                    compare_record(v.bytes(), ref)
                    seq += 1
                    want -= 1
                if views:
                    ring.release_host(views[-1].seq)
        assert moved == seq * size
        st = ring.get_stats()
        assert st.captured_records == seq and st.drained_bytes == st.captured_bytes == st.released_bytes == seq * size
        assert st.dev_ring_high_water <= dev and st.host_ring_high_water <= host
