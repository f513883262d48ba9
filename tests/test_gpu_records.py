"""Frames of many pairs per primitive in buffers with and without room for the records that the count leaves for the emit (4
bytes per primitive and bin of 4 x 4 tiles in the alternate key buffer): both give the oracle's lists, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu


def _bins(w, h):
    return ((w + 15) // 16 + 3) // 4 * (((h + 15) // 16 + 3) // 4)


def _with_records(n, bins, capacity):
    """Bytes of the alternate key buffer that the depth order, the counts and the records take (dense_layout of binsort_dense.h)."""
    up = lambda x: (x + 255) // 256 * 256
    units = min(65536 // bins, 64, n // 512, max(capacity // (bins * 2048), 12288 // bins))
    units = max(4, units // 4 * 4)
    order = up(32 * n) + 3 * up(8 * n) + up(bins * units * 64) + up(bins * units * 4)
    return order + bins * ((n + 63) // 64 * 64) * 4


def _compare(n, w, h, scale, binning, capacities):
    sc = scenes.make_scene(4, n=n, seed=n)
    sc["scale"] = np.full_like(sc["scale"], scale)
    cam = dict(scenes.make_cameras(4, w, h)[0], binning=binning)
    binned = ref.bin_sort(ref.preprocess(sc, cam), cam)
    assert binned.D >= max(32, 22 + _bins(w, h) // 30) * n and binned.D >= 1 << 18
    dev, c = B.Scene(sc), B.make_camera(cam)
    for capacity in capacities(binned.D):
        fr = B.Frame(n, w, h, int(capacity))
        fr.keys.fill_(-1)
        fr.vals.fill_(-1)
        B.render_frame(dev, c, fr)
        torch.cuda.synchronize()
        P.compare_binned(fr, binned)
        assert (fr.keys[binned.D:] == -1).all().item() and (fr.vals[binned.D:] == -1).all().item()


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n,w,h,scales", [(9000, 700, 420, (0.1, 0.12)), (9000, 1000, 700, (0.085, 0.085)), (5003, 1900, 1070, (0.06, 0.06))])
def test_both_emits(n, w, h, scales, binning):
    bins = _bins(w, h)

    def capacities(D):
        tight, roomy = D, max(2 * D, bins * n)
        assert 8 * tight < _with_records(n, bins, tight) and 8 * roomy >= _with_records(n, bins, roomy)
        return tight, roomy
    _compare(n, w, h, scales[binning], binning, capacities)


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n,w,h,scale", [(1100, 700, 420, 0.9), (4097, 333, 217, 0.4)])
def test_records_in_any_buffer(n, w, h, scale, binning):
    """Few bins, many pairs per primitive: whatever holds the pairs has the room."""
    bins = _bins(w, h)

    def capacities(D):
        assert 8 * D >= _with_records(n, bins, D)
        return D, max(2 * D, bins * n)
    _compare(n, w, h, scale, binning, capacities)
