"""The pinned ring of large copies to the host (vklb_hostcopy.hpp) on the CPU,
over a stand-in for the HIP calls it makes: sizes, a host that refuses events or
pinned memory, and calls that fail on the way."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ring_of_pinned_chunks(tmp_path):
    exe = str(tmp_path / "hostcopy_check")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                        "-I", os.path.join(ROOT, "paper_2608_04283_amd", "csrc"),
                        os.path.join(ROOT, "tests", "c", "hostcopy_check.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    for _ in range(2):  # (thread timing differs from run to run)
        r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
