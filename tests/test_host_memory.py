"""Host checks of the library's memory keeping (host_memory.h) on a stub device."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_idle_blocks_are_given_back(tmp_path):
    tests, exe = os.path.join(ROOT, "tests"), str(tmp_path / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", f"-I{tests}/hipstub",
                           f"-I{ROOT}/paper_1705_04702_amd/csrc", "-o", exe, f"{tests}/host_memory_check.cpp"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout) == (0, "ok\n")
