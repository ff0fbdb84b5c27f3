"""The library's host code on the CPU, over a stand-in for the HIP runtime
(tests/hostrt/hostrt.cpp): the order of the work that it queues on streams, what it
keeps between calls, what it does on a capturing stream, and its plans."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers not found")
    out = str(tmp_path_factory.mktemp("hostrt") / "hostrt")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__",
                        "-isystem", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2410_15240_amd", "csrc"),
                        os.path.join(ROOT, "tests", "hostrt", "hostrt.cpp"), "-o", out],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    return out


def run(exe, *args, stdin=None):
    r = subprocess.run([exe, *args], input=stdin, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    return r.returncode, r.stdout


@pytest.mark.parametrize("what", ["capture_ragged", "per_thread", "scratch_area", "tag_lanes", "ragged_plan"])
def test_host_state(exe, what):
    rc, out = run(exe, what)
    assert rc == 0 and ": 0 failures, 0 races" in out, out[-4000:]
