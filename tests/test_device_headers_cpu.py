"""Properties of the device headers over millions of random inputs, from a host build of them by g++: an entry is listed in every
4x4 cell in which a pixel reaches alpha >= 1/255 (a missed one is a wrong pixel) and in few others, a row of tiles counted
from its ends has the tiles that asking them all gives, every tile is taken once by the compositing kernels' workgroups."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_cells_rows_and_work(tmp_path):
    here, exe = os.path.join(ROOT, "tests", "host"), str(tmp_path / "headers_driver")
    # contraction off as in the projection's and binning's translation units; where the compositing kernels may contract, the
    # headers say fmaf
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wall", "-Wno-unknown-pragmas", "-Wno-unused-function",
                           "-I", here, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2503_21364_amd", "csrc"),
                           "-o", exe, os.path.join(here, "headers_driver.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and "headers driver done" in r.stdout, r.stdout[-2000:]
