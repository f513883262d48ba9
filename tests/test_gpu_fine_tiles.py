"""The compositing kernels' two forms: tiles of small images, and in images of up to 2048 tiles those with a 256th of the
frame's pairs, are walked by a wavefront per 4x4 cell, the others by one per four cells.  Images at the sizes where that
changes, with a few very long lists among short ones, and needles, whose cells are hardest to tell; image and
gradients against the oracle, to the tolerances of the other parity tests."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P
from test_gpu_backward import _compare

pytestmark = pytest.mark.gpu


def _scene(n, seed, needles):
    sc = scenes.make_scene(0, n=n, seed=seed)
    hot = np.arange(n) % 2 == 0                                 # half of them in a corner: lists of hundreds there
    sc["mean"][:2, hot] = np.float32(0.5) + np.float32(0.04) * sc["mean"][:2, hot]
    sc["opacity"] = np.where(hot, np.float32(0.05) * sc["opacity"], sc["opacity"]).astype(np.float32)
    if needles:
        sc["scale"][0] *= np.float32(3.0)
        sc["scale"][1:] *= np.float32(0.2)
    return sc


@pytest.mark.parametrize("needles", [False, True])
@pytest.mark.parametrize("w,h", [
    (256, 256),         # 256 tiles: all of them by cells
    (270, 251),         # 272, cut at both edges: those with a 256th of the pairs
    (1024, 512),        # 2048: the same
    (1024, 521),        # 2112: none
])
def test_image_and_gradients(w, h, needles):
    sc = _scene(3001, w + h, needles)
    cam = dict(scenes.make_cameras(0, w, h)[0], bg=np.array([0.3, 0.1, 0.2], np.float32), binning=1)
    r = P.full_compare(sc, cam)
    ranges = np.diff(P.to_np(r.gpu.tile_offsets).astype(np.int64))
    if 256 < ranges.size <= 2048:
        assert 0 < (256 * ranges >= ranges.sum()).sum() < ranges.size       # both forms in one frame
    _compare(sc, cam, 5)


def test_without_the_order_by_length():
    """A caller's frame need not have the order: small images go by cells, larger ones do not."""
    for w, h in ((128, 96), (400, 300)):
        sc = _scene(2000, 3, False)
        cam = dict(scenes.make_cameras(0, w, h)[0], binning=1)
        ofr = ref.render_frame(sc, cam)
        fr = P.gpu_frame(B.Scene(sc), cam, ofr.binned.D + 100)
        with_order = fr.out_rgb.clone(), fr.out_T.clone()
        fr = B.Frame(sc["n"], w, h, ofr.binned.D + 100, tile_order=False)
        B.render_frame(B.Scene(sc), B.make_camera(cam), fr)
        torch.cuda.synchronize()
        assert torch.equal(fr.out_rgb, with_order[0]) and torch.equal(fr.out_T, with_order[1])
        P.compare_image(fr, ofr.img, cam)
