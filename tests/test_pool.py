"""The working memory's lists, on the CPU: pool.cpp with a stand-in for the runtime."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lists(tmp_path):
    exe = tmp_path / "pool"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", f"-I{rocm}/include", "-pthread", "-o", str(exe),
           os.path.join(ROOT, "tests/pool_harness.cpp"), os.path.join(ROOT, "paper_2201_09004_amd/csrc/pool.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
