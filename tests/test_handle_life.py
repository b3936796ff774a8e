"""The life of a handle on the CPU: the host code of the C ABI in a program of its own, with a HIP runtime that stands in for the
real one and counts what is made, given back and waited for (host_handle_driver.cpp), under the sanitizers."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_events_and_pinned_blocks_of_handles(tmp_path):
    csrc = os.path.join(ROOT, "paper_2602_02987_amd", "csrc")
    exe = str(tmp_path / "host_handle")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-I/opt/rocm/include", f"-I{csrc}", f"-I{os.path.join(ROOT, 'include')}",
                           os.path.join(ROOT, "tests", "host_handle_driver.cpp"), os.path.join(csrc, "gnr_api.cpp"),
                           os.path.join(csrc, "gnr_tables.cpp"), "-o", exe, "-pthread"])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "clean" in res.stdout and "runtime error" not in res.stderr and "ERROR" not in res.stderr, \
        (res.stdout[-1500:], res.stderr[-3000:])
