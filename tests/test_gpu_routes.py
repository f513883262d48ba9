"""Which way stage 2 takes, and that both ways give the oracle's lists, bit for bit.

Frames of many pairs per primitive are put together from the depth-ordered primitives, all others from
counted and sorted pairs; the line is 22 pairs per primitive and one more for every 30 bins of 4 x 4 tiles, at
least 32, in buffers of at least 2^18 pairs.  The word that the device leaves in the scratch buffer (the sixth of the
eight in front of the last part, which no kernel uses) tells which way a frame went."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


def went_dense(fr) -> bool:
    chunks = (8 * (fr.capacity // 2048 + 2) + 255) // 256 * 256
    word = fr.scratch[fr.scratch_bytes - chunks - 256:].view(torch.int32)[5].item()
    assert word in (0, 1)
    return word == 1


def per_primitive(w, h):
    bins = ((w + 15) // 16 + 3) // 4 * (((h + 15) // 16 + 3) // 4)
    return max(32, 22 + bins // 30)


def _boxes(n, w, h, tiles, last, seed):
    """n axis-aligned splats in front of a camera that looks along z; tiles = (columns, rows) that the support rectangle of
    each covers, last = those of the last one."""
    rng = np.random.default_rng(seed)
    cam = dict(scenes.make_camera(np.eye(3, 4), (0, 0, 0), w, h, 60.0), binning=0)
    f = float(cam["fx"])
    mean, scale = [], []
    for i in range(n):
        cols, rows = tiles if i + 1 < n else last
        z = rng.uniform(2.0, 9.0)
        centre = []
        for count, size in ((cols, w), (rows, h)):          # an odd count is centred on a tile, an even one on a border
            lo, hi = (count + 1) // 2 + 1, (size // 16) - (count + 1) // 2 - 1
            centre.append(16.0 * rng.integers(lo, hi + 1) + (8.0 if count % 2 else 0.0))
        half = [8.0 * c - 4.0 for c in (cols, rows)]        # a quarter of a tile short of the next one
        var = [(x * x) / 11.09 - float(cam["lowpass"]) for x in half]
        mean.append([(centre[0] - float(cam["cx"])) * z / f, (centre[1] - float(cam["cy"])) * z / float(cam["fy"]), z])
        scale.append([np.sqrt(var[0]) * z / f, np.sqrt(var[1]) * z / f, 1e-4])
    return scenes.hand_placed_scene(mean, scale, opacity=list(rng.uniform(0.1, 0.9, n))), cam


@pytest.mark.parametrize("w,h,tiles,below", [
    (640, 360, (8, 4), (31, 1)),            # 60 bins: 32 pairs per primitive
    (1920, 1080, (13, 3), (38, 1)),         # 510: 39
    (3840, 2160, (10, 9), (89, 1)),         # 2040: 90
])
def test_the_line_in_pairs_per_primitive(w, h, tiles, below):
    n = 300
    assert tiles[0] * tiles[1] == per_primitive(w, h) == below[0] * below[1] + 1
    for last in (tiles, below):
        # J has a third column away from the axis: the off-axis part of a flat splat changes nothing but rounding
        sc, cam = _boxes(n, w, h, tiles, last, seed=w)
        pre = ref.preprocess(sc, cam)
        binned = ref.bin_sort(pre, cam)
        want = n * tiles[0] * tiles[1] - (tiles[0] * tiles[1] - last[0] * last[1])
        assert binned.D == want
        fr = P.gpu_frame(B.Scene(sc), cam, 1 << 18)
        P.compare_binned(fr, binned)
        assert went_dense(fr) == (last is tiles)


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n", [4096, 4097, 8193, 16384, 131072, 131073])
def test_the_order_of_chunks_and_merge_rounds(n, binning):
    """Primitives are sorted in chunks of up to 4096 and merged in one round up to 32 chunks, else in several, with equal
    depths and primitives that are not binned in between."""
    rng = np.random.default_rng(n)
    sc = scenes.make_scene(4, n=n, seed=n)
    sc["scale"] = np.full_like(sc["scale"], 0.8)
    sc["mean"][2] = np.where(rng.random(n) < 0.2, np.round(sc["mean"][2] * 16.0) / 16.0, sc["mean"][2])
    sc["opacity"][rng.random(n) < 0.1] = 0.0
    cam = dict(scenes.make_cameras(4, 200, 120)[0], binning=binning)
    pre = ref.preprocess(sc, cam)
    binned = ref.bin_sort(pre, cam)
    assert binned.D >= 32 * n
    fr = P.gpu_frame(B.Scene(sc), cam, binned.D + 5)
    P.compare_binned(fr, binned)
    assert went_dense(fr)


# ---- counting and sorting pairs, for frames that the other way would take as well: keys_alt at an odd multiple of
# 8 bytes rules that out
def _counting_frame(n, w, h, capacity):
    fr = B.Frame(n, w, h, capacity, want_offsets=True)
    fr.keys_alt = torch.empty(capacity + 1, dtype=torch.int64, device="cuda")[1:]
    assert fr.keys_alt.data_ptr() % 16 == 8
    fr.binned.keys_alt = fr.keys_alt.data_ptr()
    return fr


def _sizes_scene(n, seed, largest=60.0):
    rng = np.random.default_rng(seed)
    sc = scenes.make_scene(0, n=n, seed=seed)
    sc["scale"] = sc["scale"] * np.exp(rng.uniform(np.log(0.5), np.log(largest), n)).astype(np.float32)[None, :]
    return sc


def _areas(pre):
    rc = pre.rect.astype(int)
    return ((rc[:, 2] - rc[:, 0]) * (rc[:, 3] - rc[:, 1]))[pre.tiles_touched > 0]


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n,w,h", [
    (4000, 1920, 1080),         # 8160 tiles: counters in 32 KB
    (1500, 3000, 2000),         # 23500: in 128 KB
    (1000, 4096, 2304),         # 36864: every primitive is listed
])
def test_rectangles_of_every_size_class_by_counting(n, w, h, binning):
    """Rectangles walked by a lane, a wavefront and a workgroup (the switches are at 32 and 2048 tiles)."""
    sc = _sizes_scene(n, 55)
    cam = dict(scenes.make_cameras(0, w, h)[0], binning=binning)
    pre = ref.preprocess(sc, cam)
    binned = ref.bin_sort(pre, cam)
    area = _areas(pre)
    for lo, hi in ((0, 16), (16, 32), (32, 64), (1000, 2048), (2048, 1 << 22)):
        assert ((area > lo) & (area <= hi)).sum() > 10, (lo, hi)
    fr = _counting_frame(n, w, h, binned.D + 100)
    B.render_frame(B.Scene(sc), B.make_camera(cam), fr)
    torch.cuda.synchronize()
    P.compare_binned(fr, binned)
    assert not went_dense(fr)
    B.bin_sort(B.make_camera(cam), fr)                      # the counters are left clean
    torch.cuda.synchronize()
    P.compare_binned(fr, binned)


@pytest.mark.parametrize("binning", [0, 1])
def test_fewer_pairs_than_the_line_in_an_image_of_many_tiles(binning):
    """8193 to 32768 tiles, buffers with room for the other way, pairs below the line."""
    n, w, h = 3000, 2560, 1440
    sc = _sizes_scene(n, 12, largest=2.0)
    cam = dict(scenes.make_cameras(0, w, h)[0], binning=binning)
    pre = ref.preprocess(sc, cam)
    binned = ref.bin_sort(pre, cam)
    assert 8192 < (w // 16) * (h // 16) <= 32768 and (_areas(pre) > 32).sum() > 100
    assert binned.D < per_primitive(w, h) * n < 1 << 18
    fr = P.gpu_frame(B.Scene(sc), cam, 1 << 18)
    P.compare_binned(fr, binned)
    assert not went_dense(fr)


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("dense", [False, True])
def test_overflow_with_large_rectangles_and_a_retry(binning, dense):
    """More pairs than the buffers hold, with rectangles of every size: empty ranges, nothing written, and the same
    frame in larger buffers afterwards."""
    n, w, h = 4000, 1920, 1080
    sc = _sizes_scene(n, 55)
    cam = dict(scenes.make_cameras(0, w, h)[0], binning=binning)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    dev, c = B.Scene(sc), B.make_camera(cam)
    make = B.Frame if dense else _counting_frame
    small = make(n, w, h, binned.D // 2)
    small.keys.fill_(-1)
    B.render_frame(dev, c, small)
    torch.cuda.synchronize()
    assert B.read_status(small) == (binned.D, B.ERR_CAPACITY) and went_dense(small) == dense
    assert not small.tile_offsets.any().item() and (small.keys == -1).all().item() and (small.out_T == 1.0).all().item()
    fr = make(n, w, h, binned.D + 7, want_offsets=True) if dense else make(n, w, h, binned.D + 7)
    B.render_frame(dev, c, fr)
    torch.cuda.synchronize()
    P.compare_binned(fr, binned)
    assert went_dense(fr) == dense
