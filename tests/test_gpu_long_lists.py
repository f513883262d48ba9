"""Lists that one workgroup sorts in all the LDS of a compute unit: at the edges of that class (4096, 8192 and
16384 pairs) by counting and by merging, and more of them than the launch has workgroups; against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["spread", "steps", "two ends"])
@pytest.mark.parametrize("n", [4097, 8191, 8192, 8193, 16383, 16384, 16385, 32769])
def test_one_long_list(n, kind):
    rng = np.random.default_rng(n + len(kind))
    mean = np.zeros((n, 3))
    mean[:, 2] = {"spread": lambda: rng.uniform(1.0, 9.0, n),
                  "steps": lambda: 2.0 + 0.25 * rng.integers(0, 5, n),              # by merging: full buckets
                  "two ends": lambda: np.where(rng.random(n) < 0.5, rng.uniform(1.0, 1.5, n), rng.uniform(8.5, 9.0, n))}[kind]()
    sc = scenes.hand_placed_scene(mean, (0.01, 0.01, 0.01), opacity=list(rng.uniform(0.05, 0.9, n)))
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0)
    ofr = ref.render_frame(sc, cam)
    assert ofr.binned.D == n
    P.compare_binned(P.gpu_frame(B.Scene(sc), cam, n + 5), ofr.binned)


@pytest.mark.parametrize("n", [4097, 5000, 8192, 8193, 12000, 16384])
@pytest.mark.parametrize("size", [17, 20, 22, 24, 40, 70])
def test_clusters_around_the_limits(n, size):
    """Clusters of one size, whose buckets are around the fullest that are still ranked (22 on average, 24 in a quarter of the list, 64)."""
    rng = np.random.default_rng(n + size)
    mean = np.zeros((n, 3))
    mean[:, 2] = rng.permutation(2.0 + 0.01 * (np.arange(n) // size) + 1e-6 * rng.integers(0, 2, n))
    sc = scenes.hand_placed_scene(mean, (0.01, 0.01, 0.01), opacity=list(rng.uniform(0.05, 0.9, n)))
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    assert binned.D == n
    P.compare_binned(P.gpu_frame(B.Scene(sc), cam, n + 5), binned)


def test_more_long_lists_than_workgroups():
    """300 tiles of 4097 to 5000 pairs each, counted and sorted (with one pair per primitive the other way is far off)."""
    rng = np.random.default_rng(3)
    tx, ty = 20, 15
    per = rng.integers(4097, 5001, tx * ty)
    n, w, h = int(per.sum()), 16 * tx, 16 * ty
    cam = dict(scenes.make_camera(np.eye(3, 4), (0, 0, 0), w, h, 60.0), binning=0)
    tile = rng.permutation(np.repeat(np.arange(tx * ty), per))
    z = rng.uniform(2.0, 9.0, n)
    mean = np.stack([(16.0 * (tile % tx) + 8.0 - float(cam["cx"])) * z / float(cam["fx"]),
                     (16.0 * (tile // tx) + 8.0 - float(cam["cy"])) * z / float(cam["fy"]), z], 1)
    sc = scenes.hand_placed_scene(mean, (1e-4, 1e-4, 1e-4), opacity=list(rng.uniform(0.05, 0.9, n)))
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    assert binned.D == n and np.diff(binned.tile_offsets.astype(np.int64)).min() > 4096
    fr = P.gpu_frame(B.Scene(sc), cam, n + 5)
    P.compare_binned(fr, binned)
    B.bin_sort(B.make_camera(cam), fr)                      # the counters are left clean
    torch.cuda.synchronize()
    P.compare_binned(fr, binned)
