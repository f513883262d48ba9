"""A tile's image and gradients do not depend on the form of the compositing kernels that it goes by: the same tile alone in
an image, in an image where it holds nearly all pairs, and in one of so many tiles that none is given to several
workgroups."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu

SIZES = [(16, 16), (512, 512), (1024, 544)]             # 1, 1024 and 2176 tiles
BATCH = 255                                             # list entries that the gradient kernel stages at a time


def _scene_and_camera(n, seed, faint):
    """Round splats about the middle of the image's first tile, most of them wider than it."""
    rng = np.random.default_rng(seed)
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0, bg=(0.3, 0.1, 0.2))
    z = rng.uniform(4.0, 6.0, n)
    u, v = rng.uniform(4.0, 12.0, n), rng.uniform(4.0, 12.0, n)
    centres = [[(u[i] - float(cam["cx"])) * z[i] / float(cam["fx"]), (v[i] - float(cam["cy"])) * z[i] / float(cam["fy"]), z[i]]
               for i in range(n)]
    size = np.exp(rng.uniform(-1.5, 0.5, n))
    sc = scenes.hand_placed_scene(centres, [(s,) * 3 for s in size], opacity=rng.uniform(0.005, 0.02 if faint else 0.3, n),
                                  sh_dc=rng.uniform(0.0, 1.0, (n, 3)))
    return sc, cam


def _results(sc, cam, w, h, rgb, T=None):
    """(gradients, image, transmittance) of the first tile, the upstream gradient zero elsewhere."""
    n, c = sc["n"], dict(cam, width=w, height=h)
    fr = P.gpu_frame(B.Scene(sc), c, 2_000_000)
    assert B.read_status(fr)[1] == B.OK and int(fr.tile_offsets[1]) == n
    up = torch.zeros((4, h, w), dtype=torch.float32, device="cuda")
    up[:3, :16, :16] = torch.from_numpy(rgb.astype(np.float32)).cuda()
    if T is not None:
        up[3, :16, :16] = torch.from_numpy(T.astype(np.float32)).cuda()
    out = torch.empty((n, B.FEAT_STRIDE), dtype=torch.float32, device="cuda")
    B.render_backward(B.make_camera(c), fr, up[:3].contiguous(), up[3].contiguous(), out)
    torch.cuda.synchronize()
    return out.cpu().numpy()[:, :9], fr.out_rgb[:, :16, :16].cpu().numpy(), fr.out_T[:16, :16].cpu().numpy()


@pytest.mark.parametrize("n", [3, 40, BATCH])
def test_gradient_sums_are_rounded_once(n):
    """A gradient component of an entry is a sum over the tile's pixels in 64 bits, rounded once.  The upstream gradient is
    +1 left and -1 right of the tile's middle, with a little noise, so that the sums of the tile's parts are far larger than
    the whole: parts rounded to 32 bits before they meet would show.  The per-pixel terms are the same operations in every
    form as long as the list is one batch, so the results may differ by the one rounding (2^-24 of the value, on both
    sides), and by the order of the 64-bit additions (2^-53 of 256 terms' magnitudes, each at most 16^2 times the
    gradient's own scale)."""
    sc, cam = _scene_and_camera(n, n, False)
    rng = np.random.default_rng(n)
    side = np.where(np.arange(16) < 8, 1.0, -1.0)[None, None, :] + 1e-3 * rng.normal(size=(3, 16, 16))
    results = [_results(sc, cam, w, h, side) for w, h in SIZES]
    want = results[-1]
    for got in results[:-1]:
        assert np.array_equal(got[1], want[1]) and np.array_equal(got[2], want[2])
        scale = np.abs(want[0]).max(0)
        err = np.abs(got[0] - want[0])
        tol = np.maximum(np.spacing(np.abs(got[0])), np.spacing(np.abs(want[0]))) + 2.0 ** -53 * 256 * 256 * scale
        assert (err <= tol).all(), f"{(err > tol).sum()} components; the largest error {(err / tol).max():.1f} of what is allowed"


@pytest.mark.parametrize("n,faint", [
    (BATCH + 1, True), (2 * BATCH, True), (4 * BATCH, True),    # a segment a batch; the last of one entry; all four
    (4 * BATCH + 1, True), (9 * BATCH - 1, True),               # segments of two batches, of four
    (6000, False),                                              # all pixels stop long before the list ends
])
def test_long_lists_in_parts(n, faint):
    """Lists that several workgroups share by parts: against the oracle's 64 bits the gradients are no further off than
    those of a tile in one piece (the two forms round the transmittance and the colour behind a part differently; the
    root mean square over nine components of hundreds of entries agrees within a tenth unless one of them is worse)."""
    sc, cam = _scene_and_camera(n, n, faint)
    small = dict(cam, width=16, height=16)
    rng = np.random.default_rng(n)
    rgb, T = rng.normal(size=(3, 16, 16)).astype(np.float32), rng.normal(size=(16, 16)).astype(np.float32)
    ofr = ref.render_frame(sc, small)
    amb = ref.render_backward(ofr.pre, ofr.binned, small, rgb.astype(np.float64), T.astype(np.float64)).amb > 0
    assert amb.mean() < 0.2
    rgb[:, amb] = 0.0
    T[amb] = 0.0
    g = ref.render_backward(ofr.pre, ofr.binned, small, rgb.astype(np.float64), T.astype(np.float64))
    exact, scale = np.concatenate([g.mean2d, g.conic, g.opacity[None, :], g.rgb]).T, g.abs.T
    results = [_results(sc, cam, w, h, rgb, T) for w, h in SIZES]
    seen = scale > 1e-6 * scale.max(0)
    rms = []
    for got in results:
        assert np.array_equal(got[1], results[-1][1]) and np.array_equal(got[2], results[-1][2])
        err = np.abs(got[0] - exact)
        assert (err <= 2e-5 * scale + 1e-7).all()
        rms.append(np.sqrt(np.mean((err[seen] / scale[seen]) ** 2)))
    print(f"[forms] n={n}: rms error / sum of magnitudes {rms}", flush=True)
    assert max(rms[:-1]) <= 1.1 * rms[-1], rms
