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


@pytest.mark.parametrize("n,w,h", [(2_000_003, 700, 420), (5_000_001, 700, 420), (5_000_001, 2600, 1500),
                                   (2_000_003, 4096, 2304)])             # 36864 tiles: every primitive is listed
def test_large_and_in_no_order(n, w, h):
    sc = _scene(n, 7)
    cam = dict(scenes.make_cameras(1, w, h)[0], binning=1)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    P.compare_binned(P.gpu_frame(B.Scene(sc), cam, binned.D + 9), binned)


def _in_order(fr):
    """in_order() on the header of the scratch: the word of the index, pairs looked at, pairs near one another."""
    words = fr.scratch[:40].view(torch.int32).tolist()
    return words[3] != 0 or (words[8] >= 8 and 2 * words[9] > words[8])


# (2 M and 5 M are the lines of the workgroups for no order, 8192 tiles that up to which an order is looked for)
@pytest.mark.parametrize("n,w,h", [(2_000_003, 700, 420), (5_000_001, 700, 420)])
def test_large_and_in_order(n, w, h):
    """Primitives in spatial order with the index that gave it, without, and on the static route: the oracle's lists, and workgroups for
    order in all of them."""
    sc = _scene(n, 11)
    sc["opacity"][n // 2:] = 0.0                            # half of the scene: the look finds its pairs in what is left
    index = B.VoxelIndex(sc, 0.05)
    sc = index.reorder(sc)
    index.upload()
    cam = dict(scenes.make_cameras(1, w, h)[0], binning=1)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    dev, c = B.Scene(sc), B.make_camera(cam)
    for given in (index, None):
        fr = P.gpu_frame(dev, cam, binned.D + 9, index=given)
        assert _in_order(fr)
        P.compare_binned(fr, binned)
    if n <= B.STATIC_MAX_N:
        for t in (fr.keys, fr.vals, fr.tile_offsets):
            t.fill_(-1)
        B.bin_sort_static(c, fr)
        torch.cuda.synchronize()
        P.compare_binned(fr, binned)


@pytest.mark.parametrize("order,expected", [("no", False), ("runs of 10", False), ("runs of 64", False), ("voxels", True),
                                            ("all but a few culled", False)])
def test_looks_for_an_order(order, expected):
    n = 2_000_003
    rng = np.random.default_rng(3)
    sc = scenes.make_scene(1, n=n, seed=5)
    if order != "no":
        sc = B.VoxelIndex(sc, 0.5).reorder(sc)
    if order.startswith("runs"):
        run = int(order.split()[-1])
        starts = rng.permutation((n + run - 1) // run) * run
        perm = (starts[:, None] + np.arange(run)[None]).reshape(-1)
        perm = perm[perm < n]
        for k in ("mean", "scale", "rot", "sh"):
            sc[k] = np.ascontiguousarray(np.asarray(sc[k])[..., perm])
        sc["opacity"] = np.ascontiguousarray(sc["opacity"][perm])
    if order.startswith("all"):
        keep = np.zeros(n, bool)
        keep[rng.choice(n, 20, replace=False)] = True
        sc["opacity"] = np.where(keep, sc["opacity"], np.float32(0.0)).astype(np.float32)
    fr = B.Frame(n, 1000, 700, 1)
    B.preprocess(B.Scene(sc), B.make_camera(dict(scenes.make_cameras(1, 1000, 700)[0], binning=0)), fr)
    torch.cuda.synchronize()
    assert _in_order(fr) == expected
