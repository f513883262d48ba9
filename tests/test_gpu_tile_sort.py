"""The per-tile sort at the edges of its size classes (64 / 512 / 1024 threads, merges beyond 16384) for
depths that spread over the buckets, that fall into a few of them and that are all alike (then the index
decides and the merge sort takes over): one tile whose list has n pairs, against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


def _depths(kind, n, rng):
    if kind == "spread":
        return rng.uniform(1.0, 9.0, n)
    if kind == "clusters":      # a dense front, a few far behind
        return np.where(rng.random(n) < 0.97, rng.normal(2.0, 1e-3, n), rng.uniform(50.0, 5000.0, n))
    if kind == "steps":         # many equal depths: full buckets next to empty ones
        return 2.0 + 0.5 * rng.integers(0, 7, n)
    return np.full(n, 3.0)


@pytest.mark.parametrize("kind", ["spread", "clusters", "steps", "equal"])
@pytest.mark.parametrize("n", [1, 2, 63, 128, 129, 256, 257, 512, 513, 2048, 2049, 4096, 4097, 9000, 17000])
def test_one_tile(n, kind):
    rng = np.random.default_rng(n * 7 + len(kind))
    mean = np.zeros((n, 3))
    mean[:, 2] = _depths(kind, n, rng)
    sc = scenes.hand_placed_scene(mean, (0.01, 0.01, 0.01), opacity=list(rng.uniform(0.05, 0.9, n)))
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0)
    ofr = ref.render_frame(sc, cam)
    assert ofr.binned.D == n
    fr = P.gpu_frame(B.Scene(sc), cam, n + 5)
    P.compare_binned(fr, ofr.binned)


@pytest.mark.parametrize("n", [60, 200, 450, 1500, 2100, 3500, 4096])
@pytest.mark.parametrize("size", [6, 8, 17, 20, 24, 40, 70])
def test_clusters_around_the_limits(n, size):
    """Clusters of one size, whose buckets are around the fullest that are still ranked: on one side the list
    leaves for the merge sort after a quarter or all of it is counted, on the other it does not."""
    rng = np.random.default_rng(n + size)
    mean = np.zeros((n, 3))
    mean[:, 2] = rng.permutation(2.0 + 0.01 * (np.arange(n) // size) + 1e-6 * rng.integers(0, 2, n))
    sc = scenes.hand_placed_scene(mean, (0.01, 0.01, 0.01), opacity=list(rng.uniform(0.05, 0.9, n)))
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0)
    ofr = ref.render_frame(sc, cam)
    assert ofr.binned.D == n
    P.compare_binned(P.gpu_frame(B.Scene(sc), cam, n + 5), ofr.binned)


def test_many_lists_of_all_classes():
    """A frame whose tiles hold from none to several thousand pairs, primitives in random order."""
    sc = scenes.make_scene(0, n=60000, seed=8)
    sc["mean"][:, 30000:] *= np.float32(0.05)           # a dense spot
    cam = scenes.make_cameras(0, 240, 200)[0]
    ofr = ref.render_frame(sc, cam)
    lens = np.diff(ofr.binned.tile_offsets.astype(np.int64))
    assert lens.min() < 64 and lens.max() > 4096
    fr = P.gpu_frame(B.Scene(sc), cam, ofr.binned.D + 5)
    P.compare_binned(fr, ofr.binned)
