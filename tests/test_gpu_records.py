"""Frames of many pairs per primitive in buffers with and without room for the records that the count leaves for the emit (4
bytes per primitive and bin of 4 x 4 tiles in the alternate key buffer): both give the oracle's lists, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n,w,h,scale", [(1100, 700, 420, 0.9), (4097, 333, 217, 0.4), (9000, 1000, 700, 0.085), (5003, 1900, 1070, 0.06)])
def test_both_emits(n, w, h, scale, binning):
    sc = scenes.make_scene(4, n=n, seed=n)
    sc["scale"] = np.full_like(sc["scale"], scale)
    cam = dict(scenes.make_cameras(4, w, h)[0], binning=binning)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    bins = ((w + 15) // 16 + 3) // 4 * (((h + 15) // 16 + 3) // 4)
    assert binned.D >= max(32, 22 + bins // 30) * n and binned.D >= 1 << 18
    dev, c = B.Scene(sc), B.make_camera(cam)
    for capacity in (binned.D, max(2 * binned.D, bins * n)):
        fr = B.Frame(n, w, h, int(capacity))
        fr.keys.fill_(-1)
        fr.vals.fill_(-1)
        B.render_frame(dev, c, fr)
        torch.cuda.synchronize()
        P.compare_binned(fr, binned)
        assert (fr.keys[binned.D:] == -1).all().item() and (fr.vals[binned.D:] == -1).all().item()
