"""Reading weights back with several threads (csrc/host_copy.cpp), built with g++ against a stand-in for the HIP calls it makes
(tests/host_reader/hip): a stream there is a list of work that runs when somebody waits for it, so an order that
the code does not ask for shows as stale bytes.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_08837_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "host_reader")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_reader") / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-pthread", "-I", HERE, "-I", CSRC, os.path.join(HERE, "check.cpp"),
                    os.path.join(CSRC, "host_copy.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("name", ["order", "failing_copy", "no_memory_for_threads", "other_device", "two_callers",
                                  "pinned_by_caller"])
def test_host_reader(check, name):
    """order: copies come after the work before them for every kind of stream handle, hipStreamPerThread (every thread's
    own) among them.  failing_copy: an error is reported and leaves nothing in flight.
    no_memory_for_threads: a thread that cannot be had is done without, nothing is thrown.
    other_device: the calling thread's current device may be another one than at the first call.
    two_callers: two threads reading two stages of one context at a time each get theirs.
    pinned_by_caller: memory that is pinned already is written by one plain copy."""
    p = subprocess.run([check, name], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
