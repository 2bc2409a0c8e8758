"""The library's host code over a stand-in for the HIP runtime (tests/host_runtime.cpp; no GPU needed): what it waits for, what it
allocates and what it leaves behind when something fails.  The stand-in runs queued work at the latest moment a GPU may."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_runtime") / "host_runtime")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host_runtime.cpp"), os.path.join(CSRC, "snn_schedule.cpp"), "-o", exe], check=True)

    def run(name):
        got = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
        assert got.returncode == 0, f"{name}: {got.stdout}{got.stderr}"
    return run


def test_inputs_still_being_written_on_the_callers_stream(checks):
    checks("caller_stream")


@pytest.mark.parametrize("name", ["no_room_for_staging", "copy_fails"])
def test_a_failed_call_never_binds_parts_of_two_batches(checks, name):
    checks(name)


def test_every_entry_point_reports_a_kernel_that_gave_up_waiting(checks):
    checks("time_out_is_reported")


def test_contexts_whose_kernels_wait_between_workgroups_take_turns(checks):
    checks("turns")
