"""Kernel launches on the CPU: csrc/xattn_launch.h built with g++ against a stand-in for the HIP runtime
(tests/host/launch_main.cpp), with failing lookups and launches, and streams of a device that is not the current one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches(tmp_path):
    exe = os.path.join(str(tmp_path), "launch_host")
    res = subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-fsanitize=undefined",
                          "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "host", "launch_main.cpp"), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "all scenarios ran" in run.stdout, run.stdout + run.stderr
