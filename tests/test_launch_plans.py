"""How launches are planned (host runtime on the CPU stand-in, tests/cpu_runtime/): the number of workgroups follows the
rows that a keep vector is expected to keep, and what a launch reads, and out of which stretch, decides whether it does so past the memory-side
cache."""
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

    def run(src, width, reqs, each, out, mask=0, tensors=1, keep="none", step=0, every=1, indexed=0):
        p = subprocess.run([exe, *map(str, (src, width, reqs, each, out, mask, tensors, keep, step, every, indexed))], timeout=60,
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


MB = 1 << 20


@pytest.mark.parametrize("src,width,out,mask", [(BF16, 4096, FP8, 0), (BF16, 4096, BF16, 0), (FP32, 4096, 0, 7), (BF16, 4096, 0, 5),
                                                (BF16, 4096, BF16, 5), (BF16, 512, 0, 5)])
def test_past_the_cache(plan, src, width, out, mask):
    row = width * (4 if src == FP32 else 2)

    def reads(mb, **how):
        return plan(src, width, 16, mb * MB // row // 16 // how.get("tensors", 1), out, mask, **how)["read_once"]

    assert (reads(200), reads(255), reads(257), reads(400)) == (0, 0, 1, 1)
    # at least half as much out of a larger stretch
    assert (reads(126, every=4), reads(130, every=4), reads(125, every=2), reads(130, every=2), reads(90, every=30)) == (0, 1, 0, 1, 0)
    for keep in ("10" * 8, "unknown"):
        assert (reads(254, keep=keep), reads(260, keep=keep)) == (0, 1)
    assert (reads(400, keep="1" + "0" * 15), reads(800, keep="1110" + "0" * 12)) == (0, 1)
    # where that is not known, what is expected to be read: of a launch with a keep vector not what is listed
    assert (reads(255, indexed=1), reads(257, indexed=1), reads(100, every=4, indexed=1)) == (0, 1, 0)
    half = dict(indexed=1, keep="10" * 8)
    assert (reads(400, **half), reads(500, **half), reads(520, **half)) == (0, 0, 1)
    assert (reads(1600, indexed=1, keep="1" + "0" * 15), reads(270, indexed=1, keep="1" * 16)) == (0, 1)
    assert (reads(400, indexed=1, keep="unknown"), reads(520, indexed=1, keep="unknown")) == (0, 1)
    # a batch of rows that a wavefront or more takes: from half of the cache on
    early = int(width != 512)
    assert (reads(127, tensors=8), reads(128, tensors=8), reads(260, tensors=8)) == (0, early, 1)


@pytest.mark.parametrize("out,least", [(BF16, (72, 80)), (2, (80, 104)), (FP8, (104, 136))])
def test_short_steps_of_large_launches_are_dealt_flat(plan, out, least):
    def rows_kernel(units, rows, ragged):
        return plan(BF16, 8 * units, 50 if ragged else 250, rows // 50 if ragged else 1, out, tensors=1 if ragged else rows // 250)["rows_kernel"]

    for ragged in (0, 1):
        at = least[ragged]
        for parts in (1, 2, 3):                     # steps per row
            if parts > 1 and at * parts <= 256 * (parts - 1):
                continue
            assert rows_kernel(at * parts, 25000, ragged) == 1 and rows_kernel(at * parts - 1, 25000, ragged) == 0
        assert rows_kernel(64, 11500, ragged) == 1 and rows_kernel(64, 12250, ragged) == 0
        assert rows_kernel(63, 1000, ragged) == 0 and rows_kernel(256, 100000, ragged) == 1


@pytest.mark.parametrize("out", [BF16, FP8])
@pytest.mark.parametrize("tensors", [1, 2, 8, 16])
def test_batches_of_short_rows_dealt_flat(plan, out, tensors):
    """Shared evenly among five workgroups per compute unit, beyond nine rounds of a batch two items each, beyond twenty four."""
    for rounds in (1, 2, 4, 5, 8, 9, 10, 20, 21, 40):
        each = (rounds * 1280 * 32 - 1600) // tensors // 50     # rows of 32 units, 32 to an item
        items = -(-(-(-50 * each * 32 // 256)) // 4)
        share = rounds if tensors == 1 or rounds <= 9 else 2 if rounds <= 20 else 4
        assert -(-items * tensors // 1280) == rounds
        got = plan(BF16, 256, 50, each, out, tensors=tensors)
        assert got["rows_kernel"] == 0 and got["grid"] == (items if rounds == 1 else -(-items // share))


@pytest.mark.parametrize("src,elems,rows", [(BF16, 1024, 132000), (BF16, 256, 530000), (2, 1000, 135000), (FP32, 512, 132000), (BF16, 2040, 66500)])
def test_statistics_of_short_rows_past_the_cache(plan, src, elems, rows):
    """What tests/test_gpu_row_routes.py compares with the oracle takes the variant it is about."""
    p = plan(src, elems, 40, rows // 40 - 1, 0, 7)
    assert p["read_once"] == 1 and p["rows_kernel"] == int(elems * (4 if src == FP32 else 2) // 16 >= 192)
