"""The serving form's host side against a pretended device (no GPU): a lost
request leaves its slot usable, and a request in flight does not hold a host
core."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("serve") / "serve_host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-Wno-subobject-linkage", "-pthread",
                    "-o", exe, os.path.join(HERE, "native", "serve_host.cpp")], check=True)
    return lambda what: subprocess.run([exe, what], capture_output=True, text=True, timeout=60,
                                       check=True).stdout.splitlines()


def test_slot_of_a_lost_request(program):
    """A request of which only 5 of 8 blocks finish fails; the next ones on its
    slot end with their own last block, with all of their own bins."""
    first, lost, *after = program("lost")
    assert first == "0" and lost == "3"          # OSC_OK, OSC_ERR_DEVICE
    assert after == ["0 0 1 2 3 4 5 6 7"] * 2


def test_cpu_time_while_a_request_runs(program):
    """Half a second of one request in flight costs the process well under half
    of a core (0.2 with sleeps of 20 us; 0.64 where it also watches between
    them)."""
    status, share = program("idle")[0].split()
    assert status == "0" and float(share) < 0.4
