"""The tiles of a bin that a splat surely keeps and those that have to be asked (tile_test.h), from a host build by g++, against
asking every tile, over millions of random ellipses."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bin_tiles(tmp_path):
    here, exe = os.path.join(ROOT, "tests", "host"), str(tmp_path / "bin_tiles_driver")
    # contraction off as in the binning's translation unit
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wall", "-Wno-unknown-pragmas", "-Wno-unused-function",
                           "-I", here, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2503_21364_amd", "csrc"),
                           "-o", exe, os.path.join(here, "bin_tiles_driver.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and "bin tiles driver done" in r.stdout, r.stdout[-2000:]
