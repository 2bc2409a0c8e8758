"""The library's host code over a stand-in for the HIP runtime (tests/host_runtime.cpp; no GPU needed): what it waits for, what it
allocates and what it leaves behind when something fails.  The stand-in runs queued work at the latest moment a GPU may."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")


def _build(folder, *flags):
    exe = str(folder / "host_runtime")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-pthread", *flags, "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                    "/opt/rocm/include", os.path.join(ROOT, "tests", "host_runtime.cpp"), os.path.join(CSRC, "snn_schedule.cpp"),
                    "-o", exe], check=True)

    def run(name):
        got = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
        if "unexpected memory mapping" in got.stderr:
            pytest.skip("the thread sanitizer cannot start on this kernel")
        assert got.returncode == 0, f"{name}: {got.stdout}{got.stderr[:2000]}"
    return run


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("host_runtime"))


@pytest.fixture(scope="module")
def thread_checks(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("host_runtime_threads"), "-fsanitize=thread")


def test_inputs_still_being_written_on_the_callers_stream(checks):
    checks("caller_stream")


@pytest.mark.parametrize("name", ["no_room_for_staging", "copy_fails"])
def test_a_failed_call_never_binds_parts_of_two_batches(checks, name):
    checks(name)


def test_every_entry_point_reports_a_kernel_that_gave_up_waiting(checks):
    checks("time_out_is_reported")


def test_contexts_whose_kernels_wait_between_workgroups_take_turns(thread_checks):
    thread_checks("turns")


def test_contexts_of_several_threads_share_no_exchange_buffer(thread_checks):
    thread_checks("blocks")


def test_workspace_is_allocated_once(checks):
    checks("workspace")


def test_activity_follows_every_call(checks):
    checks("rates")


def test_gradients_do_not_follow_the_memory_that_is_free(checks):
    checks("split_room")


def test_workspace_of_the_weight_gradients_is_part_of_the_step(checks):
    checks("split_workspace")


def test_exchange_of_the_forward_part_by_column_holds_the_longest_tile(checks):
    checks("column_places")


def test_form_by_column_only_where_it_can_be_used(checks):
    checks("column_form")
