"""Stage 2 with counting workgroups of every size (512 to 8192 primitives, by the number of primitives and by whether the
projection had an index), on both sides of every line, ragged last workgroups, groups without a pair in between; against the oracle."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    rng = np.random.default_rng(seed)
    sc = scenes.make_scene(1, n=n, seed=seed)
    sc["scale"] = (sc["scale"] * np.exp(rng.uniform(-0.5, 1.5, n))).astype(np.float32)       # some rectangles beyond 32 tiles
    sc["opacity"][rng.random(n) < min(0.95, n / 3e5)] = 0.0
    sc["opacity"][n // 3:n // 3 + min(n // 4, 20000)] = 0.0                               # whole workgroups without a pair
    return sc


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("n", [511, 513, 65536, 65537, 131072, 131073, 262145])
def test_by_number_and_order(n, ordered):
    sc, index = _scene(n, n), None
    if ordered:
        index = B.VoxelIndex(sc, 1.0)
        sc = index.reorder(sc)
        index.upload()
    for binning in (0, 1):
        cam = dict(scenes.make_cameras(1, 700, 420)[0], binning=binning)
        binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
        fr = P.gpu_frame(B.Scene(sc), cam, binned.D + 9, index=index)
        P.compare_binned(fr, binned)
        B.bin_sort(B.make_camera(cam), fr)                  # the counters are left clean
        torch.cuda.synchronize()
        P.compare_binned(fr, binned)


@pytest.mark.parametrize("n,w,h", [(2_000_003, 700, 420), (5_000_001, 700, 420), (5_000_001, 2600, 1500)])
def test_large_and_in_no_order(n, w, h):
    sc = _scene(n, 7)
    cam = dict(scenes.make_cameras(1, w, h)[0], binning=1)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    P.compare_binned(P.gpu_frame(B.Scene(sc), cam, binned.D + 9), binned)
