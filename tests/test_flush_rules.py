"""Where the copy of a flush goes, and what drains and polls report while one is under way: the host
runtime on the CPU stand-in (tests/cpu_runtime/), one scenario of flush_rules_driver.cpp per test."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CPU = os.path.join(ROOT, "tests", "cpu_runtime")
CSRC = os.path.join(ROOT, "paper_2605_11093_amd", "csrc")

SCENARIOS = ["waiting_drain_after_a_flush_that_gave_up", "polling_alone_sees_a_flush_that_gave_up",
             "captured_records_do_not_wait_for_work_behind_them",
             "records_with_a_probe_do_not_wait_for_work_behind_it",
             "a_flush_that_gives_up_delivers_what_was_captured",
             "a_flush_that_gives_up_delivers_what_gets_captured",
             "a_flush_that_gives_up_leaves_room_to_the_producer",
             "an_unanswered_capture_query_leaves_no_error",
             "spans_up_to_the_limit_go_behind_the_captures",
             "other_rings_and_spans_do_not_go_behind_the_captures",
             "other_threads_flushes_stay_off_the_producers_stream",
             "noted_records_do_not_wait_for_the_captures_behind_them",
             "a_small_noted_part_goes_with_the_rest", "a_batch_in_two_launches",
             "commit_slots_wait_for_a_flush_that_gave_up", "a_failing_gpu_is_not_a_flush_that_takes_long",
             "a_flush_does_not_give_up_on_its_own_copy",
             "the_last_copy_leaves_the_compute_units_to_work_behind_the_captures",
             "a_captured_stream_is_not_asked_for_its_state",
             "other_drains_do_not_copy_by_notes", "a_flush_leaves_an_open_step_alone",
             "a_step_destroyed_while_open_is_not_drained_by_its_notes",
             "a_batch_goes_by_two_launches_only_for_flushes_that_copy_by_notes",
             "where_the_batches_of_the_gpu_test_are_cut",
             "a_ring_that_drains_by_kernel_copies_behind_the_captures",
             "the_rest_of_a_long_copy_stays_with_its_engine"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("flush_rules") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address", "-pthread",
           "-I", CPU, "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", exe]
    for src in [os.path.join(CSRC, f) for f in ("dmi_host.hip", "dmi_step.hip", "dmi_exporter.hip")] + \
            [os.path.join(CPU, f) for f in ("fake_hip.cpp", "cpu_kernels.cpp", "flush_rules_driver.cpp")]:
        cmd += ["-x", "c++", src]
    subprocess.check_call(cmd)
    return exe


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_flush(driver, scenario):
    p = subprocess.run([driver, scenario], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=60,
                       env=dict(os.environ, ASAN_OPTIONS="exitcode=67"))
    assert p.returncode == 0, p.stdout.decode(errors="replace")[-4000:]
