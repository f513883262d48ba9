"""The counting workgroups of stage 2 (lmk_gs_internal.h), from a host build by g++: each primitive belongs to one of them, on both
sides of every line of their size and up to the largest number of primitives."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bin_share(tmp_path):
    here, exe = os.path.join(ROOT, "tests", "host"), str(tmp_path / "bin_share_driver")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-Wno-unused-function",
                           "-I", here, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2503_21364_amd", "csrc"),
                           "-o", exe, os.path.join(here, "bin_share_driver.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and "bin share driver done" in r.stdout, r.stdout[-2000:]
