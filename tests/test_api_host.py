"""The C-ABI layer's workspaces and splits on the CPU: csrc/xattn_api.cpp built with g++ against a stand-in for the
HIP runtime and the launches (tests/host/api_main.cpp), with failing allocations and streams under capture."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_14686_amd", "csrc")
SOURCES = [os.path.join(ROOT, "tests", "host", "api_main.cpp")] + \
    [os.path.join(CSRC, f) for f in ("xattn_api.cpp", "xattn_error.cpp")]


def test_workspaces_and_splits(tmp_path):
    exe = os.path.join(str(tmp_path), "api_host")
    res = subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-pthread", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                          "-fsanitize=undefined", "-fno-sanitize-recover=all"] + SOURCES + ["-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "all scenarios ran" in run.stdout, run.stdout + run.stderr
