"""What a drain kernel copies, piece by piece: rings that end on the way, spans of more bytes than one launch takes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CPU = os.path.join(ROOT, "tests", "cpu_runtime")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_spans_lie_where_the_stream_says(tmp_path):
    exe = str(tmp_path / "spans")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CPU,
                           "-I", os.path.join(ROOT, "paper_2605_11093_amd", "csrc"), "-o", exe,
                           os.path.join(CPU, "spans_driver.cpp")])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=60)
    assert p.returncode == 0, p.stdout.decode(errors="replace")
