"""The projection where wavefronts are partly alive: tiles of small rectangles tested in a row, outputs written in whole
lines; against the oracle, and nothing behind the last primitive is touched."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alive", [0.02, 0.3, 0.7, 1.0])
@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 63, 65, 257, 1000])
def test_partly_alive_wavefronts(n, degree, alive):
    rng = np.random.default_rng(n + 10 * degree)
    sc = scenes.make_scene(0, n=n, seed=n)
    sc["scale"] = (sc["scale"] * np.exp(rng.uniform(-1.0, 2.2, n))).astype(np.float32)      # 1 to some dozen tiles
    sc["opacity"][rng.random(n) >= alive] = 0.0
    sc["sh_degree"] = degree
    for binning in (0, 1):
        cam = dict(scenes.make_cameras(0, 500, 300)[0], binning=binning)
        pre = ref.preprocess(sc, cam)
        fr = B.Frame(n + 64, 500, 300, 16)
        guards = [fr.depth, fr.tiles_touched, fr.rect, fr.feat]
        for t in guards:
            t.view(torch.uint8).fill_(0x5a)
        B.preprocess(B.Scene(sc), B.make_camera(cam), fr)
        torch.cuda.synchronize()
        P.compare_projected(fr, pre)
        assert all((t[n:].contiguous().view(torch.uint8) == 0x5a).all().item() for t in guards)


@pytest.mark.parametrize("degree", [1, 3])
@pytest.mark.parametrize("w,h,spread", [(700, 420, 1.0), (1900, 1070, 1.6), (4000, 300, 1.6)])
def test_rectangles_around_the_rows(w, h, spread, degree):
    """Rectangles of up to and of more than 128 tiles, from where on a lane counts a row of tiles, needles among them."""
    n = 1500
    rng = np.random.default_rng(w)
    sc = scenes.make_scene(0, n=n, seed=w)
    sc["scale"] = (sc["scale"] * np.exp(rng.uniform(1.0, 1.5 + 2.0 * spread, n))).astype(np.float32)
    sc["scale"][:2, rng.random(n) < 0.3] *= np.float32(0.01)
    sc["sh_degree"] = degree
    cam = dict(scenes.make_cameras(0, w, h)[0], binning=1)
    pre = ref.preprocess(sc, cam)
    rc = pre.rect.astype(int)
    area = ((rc[:, 2] - rc[:, 0]) * (rc[:, 3] - rc[:, 1]))[pre.tiles_touched > 0]
    assert (area <= 64).sum() > 30 and ((area > 64) & (area <= 128)).sum() > 30 and ((area > 128) & (area <= 512)).sum() > 30 and (area > 512).sum() > 10
    fr = B.Frame(n, w, h, 16)
    B.preprocess(B.Scene(sc), B.make_camera(cam), fr)
    torch.cuda.synchronize()
    P.compare_projected(fr, pre)
