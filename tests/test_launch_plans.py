"""How launches are planned (host runtime on the CPU stand-in, tests/cpu_runtime/): the number of workgroups follows the
rows that a keep vector is expected to keep."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CPU = os.path.join(ROOT, "tests", "cpu_runtime")
CSRC = os.path.join(ROOT, "paper_2605_11093_amd", "csrc")
BF16, FP32, FP8 = 1, 3, 4
FULL = 8 * 256          # workgroups that fill the GPU


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("plans") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-pthread", "-I", CPU, "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), "-o", exe]
    for src in [os.path.join(CSRC, f) for f in ("dmi_host.hip", "dmi_step.hip", "dmi_exporter.hip")] + \
            [os.path.join(CPU, f) for f in ("fake_hip.cpp", "cpu_kernels.cpp", "plan_driver.cpp")]:
        cmd += ["-x", "c++", src]
    subprocess.check_call(cmd)

    def run(src, width, reqs, each, out, mask=0, tensors=1, keep="none", step=0):
        p = subprocess.run([exe, *map(str, (src, width, reqs, each, out, mask, tensors, keep, step))], timeout=60,
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, env=dict(os.environ, ASAN_OPTIONS="exitcode=67"))
        assert p.returncode == 0, p.stdout.decode(errors="replace")[-4000:]
        return {k: int(v) for k, v in (f.split("=") for f in p.stdout.decode().split())}
    return run


# a launch's workgroups for that many rows: a workgroup per row; a wavefront per row; a wavefront per 256 units
PER_ROWS = {"workgroup": ((FP32, 4096, 0, 7), lambda r: r), "wavefront": ((BF16, 1536, 0, 5), lambda r: (r + 3) // 4),
            "units": ((BF16, 4096, FP8, 0), lambda r: (2 * r + 3) // 4)}


@pytest.mark.parametrize("how", [*PER_ROWS])
@pytest.mark.parametrize("each", [1, 4, 60, 1000])
@pytest.mark.parametrize("tensors", [1, 8])
def test_keep_vectors(plan, how, each, tensors):
    (src, width, out, mask), groups = PER_ROWS[how]
    ask = dict(src=src, width=width, reqs=16, each=each, out=out, mask=mask, tensors=tensors)
    everything = plan(**ask)
    assert everything["grid"] == groups(16 * each) or everything["decode"]
    # the host knows the vector: as many workgroups as without one for those rows
    for kept in (1, 3, 8, 16):
        assert plan(**ask, keep="1" * kept + "0" * (16 - kept))["grid"] == groups(kept * each)
    # it does not (or the vector changes between replays): enough to fill the GPU, if there are rows for that; half of the rows
    want = max(groups(8 * each), min(groups(16 * each), -(-FULL // tensors)))
    assert plan(**ask, keep="unknown")["grid"] == want
    assert plan(**ask, keep="1" * 16, step=1)["grid"] == want
