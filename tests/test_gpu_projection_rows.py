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
