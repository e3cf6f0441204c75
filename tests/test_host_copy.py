"""The host side of the transfers between caller-owned arrays and the device
(transfer.hpp) on the CPU, with stand-ins for the runtime calls."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1909_13772_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include/hip/hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path_factory.mktemp("host_copy") / "host_copy_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
           "-I" + CSRC, os.path.join(HERE, "host_copy_check.cpp"), "-o", exe]
    b = subprocess.run(cmd, capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip() == "ok", (what, r.stdout[-500:], r.stderr[-2000:])

    return run


def test_copies_are_enqueued_by_the_calling_thread(check):
    """The bound stream may be the calling thread's own: nothing is enqueued
    from the copying threads, and every array arrives whole."""
    check("round_trips")


def test_no_exception_without_memory(check):
    """With every host allocation failing (the lists, the threads) nothing is
    thrown through the C entry points: the calling thread does the work."""
    check("no_memory")


def test_streams_of_another_device(check):
    """The caller's current device need not be the bound stream's: events
    belong to the stream's device, and the current one stays."""
    check("devices")


def test_pinned_arrays_are_copied_in_place(check):
    """Arrays that the runtime knows go over the link as they are."""
    check("known_memory")


def test_small_transfers_take_no_buffers(check):
    check("small_transfers")


def test_pinned_buffers_are_shared_and_bounded(check):
    """Handles cost no pinned memory, transfers in turn share one buffer, at
    most two are kept, none outlives the last handle, and none goes back while
    a stream may still use it."""
    check("pool")


def test_a_failed_transfer_waits_for_the_stream(check):
    """After an error nothing still reads or writes the caller's arrays."""
    check("early_end")
