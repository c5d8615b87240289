"""The workspace kept between template builds, on a pretended device (no GPU):
it never costs the library an allocation, and ends with its context."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_build_workspace_gives_way(tmp_path):
    exe = str(tmp_path / "memory_host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-Wno-subobject-linkage", "-pthread",
                    "-o", exe, os.path.join(HERE, "native", "memory_host.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout
    assert out.splitlines() == [
        "builds 0 0 0", "kept 500 300 400",
        "binned 0", "kept 0 0 400",              # both workspaces of that device
        "build 0", "fill 0", "kept 0 0 400",
        "build 0", "held 0", "binned 2", "same 1",   # OSC_ERR_OUT_OF_MEMORY, nothing freed
        "fill 0", "left 0"]
