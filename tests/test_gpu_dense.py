"""Stage 2 of frames with very many pairs per primitive (the primitives are put into depth order once
and every tile's list is written front to back): keys, values and ranges against the oracle, bit for
bit.  Taken when the buffers hold 2^18 pairs and, in images of up to 300 bins, 32 per primitive, and the
frame has 32 per primitive (the line itself, larger images and the merge rounds: test_gpu_routes.py); the cases
are images whose bins of 4 x 4 tiles are cut at the edges, few and many primitives, and a frame below the line."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu

CAP = 1 << 22


def _scene(n, seed, mul, flat=False):
    sc = scenes.make_scene(4, n=n, seed=seed)
    sc["scale"] = sc["scale"] * np.float32(mul)
    if flat:                                   # one depth for many: the index decides the order
        sc["mean"][2] = np.where(np.arange(n) % 3 > 0, np.float32(0.25), sc["mean"][2])
    return sc


@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("n,w,h,mul,flat,dense", [
    (1, 512, 512, 8.0, False, True),           # one primitive
    (65, 640, 360, 4.0, False, True),          # a unit and a bit
    (3000, 1000, 500, 2.0, False, True),       # 63 x 32 tiles: bins cut on the right
    (5000, 777, 1031, 1.0, True, True),        # bins cut on both sides, equal depths
    (20000, 640, 360, 1.0, False, True),
    (20000, 640, 360, 0.05, False, False),     # the buffers allow it, the frame has few pairs
])
def test_lists_equal_the_oracle(n, w, h, mul, flat, dense, binning):
    sc = _scene(n, 17 + n, mul, flat)
    cam = dict(scenes.make_cameras(4, w, h)[0], binning=binning)
    ofr = ref.render_frame(sc, cam)
    assert (ofr.binned.D >= 32 * n) == dense, (ofr.binned.D, n)
    cap = max(CAP, ofr.binned.D + 100)
    dev = B.Scene(sc)
    fr = P.gpu_frame(dev, cam, cap)
    P.compare_binned(fr, ofr.binned)
    P.compare_image(fr, ofr.img, cam)
    # again on the same buffers
    B.bin_sort(B.make_camera(cam), fr)
    torch.cuda.synchronize()
    P.compare_binned(fr, ofr.binned)


def test_culled_primitives_and_the_fixed_scratch_array():
    sc = _scene(4000, 5, 2.0)
    sc["mean"][2, ::2] += np.float32(50.0)      # behind the camera
    sc["opacity"][1::4] = 0.0
    cam = dict(scenes.make_cameras(4, 800, 600)[0], binning=1)
    ofr = ref.render_frame(sc, cam)
    assert ofr.binned.D >= 32 * sc["n"]
    fr = P.gpu_frame(B.Scene(sc), cam, CAP)
    P.compare_binned(fr, ofr.binned)
    fr.keys.fill_(-1); fr.vals.fill_(-1); fr.tile_offsets.fill_(-1)
    status = torch.zeros(2, dtype=torch.int64, device="cuda")
    B.bin_sort_static(B.make_camera(cam), fr, status)
    torch.cuda.synchronize()
    assert status.tolist() == [ofr.binned.D, 0]
    P.compare_binned(fr, ofr.binned)


def test_overflow_leaves_empty_ranges():
    sc = _scene(20000, 6, 6.0)
    cam = dict(scenes.make_cameras(4, 1920, 1080)[0], binning=0)
    dev = B.Scene(sc)
    fr = B.Frame(dev.n, 1920, 1080, CAP)
    fr.keys.fill_(-1)
    B.render_frame(dev, B.make_camera(cam), fr)
    torch.cuda.synchronize()
    D, status = B.read_status(fr)
    assert D > CAP and status == B.ERR_CAPACITY
    assert not fr.tile_offsets.any().item() and (fr.keys == -1).all().item()
    assert (fr.out_T == 1.0).all().item()


def test_lists_of_fewer_pairs_than_the_projection_counted():
    """Primitives taken out (tiles_touched = 0) between the projection and stage 2: the frame's pair count that decides how the
    depth order is shared out is then larger than what the lists add up to, and the emit has to go by the same one as the count.
    The lists are those of the scene without them."""
    n, w, h = 100_000, 1920, 1080
    bins = 30 * 17
    sc = scenes.make_scene(4, n=n, seed=3)
    sc["scale"] = np.full_like(sc["scale"], 0.16)
    out = np.random.default_rng(5).random(n) < 0.5
    rest = dict(sc, opacity=np.where(out, np.float32(0.0), sc["opacity"]))
    cam = B.make_camera(dict(scenes.make_cameras(4, w, h)[0], binning=0))
    probe = B.Frame(n, w, h, 1)
    B.preprocess(B.Scene(sc), cam, probe)
    D = int(probe.tiles_touched.sum().item())
    a, b = B.Frame(n, w, h, D), B.Frame(n, w, h, D)
    B.preprocess(B.Scene(sc), cam, a)
    a.tiles_touched[torch.from_numpy(out).cuda()] = 0
    B.bin_sort(cam, a)
    B.preprocess(B.Scene(rest), cam, b)
    B.bin_sort(cam, b)
    torch.cuda.synchronize()
    kept, status = B.read_status(a)
    assert (kept, status) == B.read_status(b) and status == B.OK
    assert D // (bins * 2048) >= kept // (bins * 2048) + 8 and D >= 40 * n          # not shared out alike
    assert torch.equal(a.tile_offsets, b.tile_offsets)
    assert torch.equal(a.keys[:kept], b.keys[:kept]) and torch.equal(a.vals[:kept], b.vals[:kept])
