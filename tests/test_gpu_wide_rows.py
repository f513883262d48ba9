"""Rectangles of more than 128 tiles under the tile test: the projection counts a row of tiles from where two ellipses cross
it and asks those in between.  Round splats, ellipses and needles of every direction, axis-parallel and nearly so, that cover, cross, touch or
miss the edges of a large image: tiles kept per primitive and the sorted lists against the oracle, exactly."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["round", "ellipse", "needle", "axis", "nearly"])
@pytest.mark.parametrize("w,h", [(2560, 1440), (1100, 4100)])       # rows beyond the 64 lanes of a wavefront in the second
def test_tiles_kept(w, h, kind):
    n = 400
    sc = scenes.make_scene(4, n=n, seed=len(kind) + w)
    rng = np.random.default_rng(7)
    long, short = np.exp(rng.normal(0.2, 0.8, n)), np.exp(rng.normal(-4.0, 1.0, n))
    third = dict(round=long, ellipse=0.2 * long).get(kind, short)
    sc["scale"] = np.stack([long, third, third]).astype(np.float32)
    if kind in ("axis", "nearly"):
        angle = np.pi / 2 * rng.integers(0, 2, n) + (0.0 if kind == "axis" else rng.choice([1e-2, 1e-3, 1e-4], n))
        sc["rot"] = np.stack([np.cos(angle / 2), 0 * angle, 0 * angle, np.sin(angle / 2)]).astype(np.float32)
    cam = dict(scenes.make_cameras(4, w, h)[0], binning=1)
    ofr = ref.render_frame(sc, cam)
    r = ofr.pre.rect.astype(np.int64)
    area = (r[:, 2] - r[:, 0]) * (r[:, 3] - r[:, 1])
    assert (area[ofr.pre.tiles_touched > 0] > 512).sum() > n // 20
    fr = P.gpu_frame(B.Scene(sc), cam, ofr.binned.D + 100)
    P.compare_projected(fr, ofr.pre)
    P.compare_binned(fr, ofr.binned)
