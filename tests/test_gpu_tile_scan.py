"""Ranges and order of the tiles at the edges of the scan's chunks (8192 tiles, four of them, more), against the oracle; the order
is a permutation by falling power of two of the list length."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(2048, 1024), (2049, 1024), (2048, 2048), (2048, 2049), (4096, 1536), (4096, 2047), (4096, 2048), (4096, 2049)])
def test_chunks_of_tiles(w, h):
    n = 3000
    sc = scenes.make_scene(0, n=n, seed=w + h)
    cam = dict(scenes.make_cameras(0, w, h)[0], binning=1)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    fr = P.gpu_frame(B.Scene(sc), cam, binned.D + 5)
    P.compare_binned(fr, binned)
    order = fr.tile_order.cpu().numpy()
    lens = np.diff(binned.tile_offsets.astype(np.int64))
    assert np.array_equal(np.sort(order), np.arange(lens.size))
    bucket = np.ceil(np.log2(np.maximum(lens, 1)))[order]
    assert (np.diff(bucket) <= 0).all()
    fr2 = B.Frame(n, w, h, max(binned.D // 2, 1))           # too small: every range is empty
    B.render_frame(B.Scene(sc), B.make_camera(cam), fr2)
    torch.cuda.synchronize()
    assert B.read_status(fr2) == (binned.D, B.ERR_CAPACITY) and not fr2.tile_offsets.any().item()
