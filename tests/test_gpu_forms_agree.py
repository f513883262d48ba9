"""A tile's image and gradients do not depend on the form of the compositing kernels that it goes by: the same tile alone in
an image, in an image where it holds nearly all pairs, and in one of so many tiles that none is given to several
workgroups."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_21364_amd import binding as B, scenes
import parity as P
from test_gpu_backward import _compare

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


# ---------------------------------------------------------------- values that are not finite
# float atomics in any order: a few 2^-24 of the sum of up to 256 terms' magnitudes
SAME = dict(rtol=1e-5, atol=1e-5)
FRONT, FAINT, SPOT, BACK = range(4)


def _layers(fillers):
    """FRONT and BACK cover the tile, and between them `fillers` faint entries do, half in front of FAINT and SPOT and half
    behind.  FAINT sits between four pixel centres of the first cell and reaches 1/255 at none of them, SPOT lies in
    another cell of that 8x8 block."""
    cam = scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0)
    at = lambda u, v, z: [(u - float(cam["cx"])) * z / float(cam["fx"]), (v - float(cam["cy"])) * z / float(cam["fy"]), z]
    depths = np.concatenate([np.linspace(4.1, 4.9, fillers // 2), np.linspace(5.6, 5.9, fillers - fillers // 2)])
    sc = scenes.hand_placed_scene([at(8, 8, 4.0), at(2, 2, 5.0), at(6, 6, 5.5), at(8, 8, 6.0)] + [at(8, 8, z) for z in depths],
                                  [(5.0,) * 3, (1e-4,) * 3, (1e-4,) * 3, (5.0,) * 3] + [(5.0,) * 3] * fillers,
                                  opacity=[0.3, 0.0085, 0.5, 0.4] + [0.01] * fillers,
                                  sh_dc=[(0.4,) * 3, (0.5,) * 3, (0.8,) * 3, (0.2,) * 3] + [(0.3,) * 3] * fillers)
    early = np.concatenate([[True, False, False, False], depths < 5.0])
    late = np.concatenate([[False, False, False, True], depths > 5.0])
    return sc, cam, early, late


def _layer_grads(sc, cam, w, h, pixel=None, colour=None):
    """Gradients of the entries for an upstream gradient on the first tile, `pixel` = (plane, value) at (1, 1) of
    it, `colour` = (entry, value)."""
    c = dict(cam, width=w, height=h)
    fr = P.gpu_frame(B.Scene(sc), c, 2_000_000)
    assert B.read_status(fr)[1] == B.OK and int(fr.tile_offsets[1]) == sc["n"]
    rng = np.random.default_rng(3)
    up = torch.zeros((4, h, w), dtype=torch.float32, device="cuda")
    up[:, :16, :16] = torch.from_numpy(rng.normal(size=(4, 16, 16)).astype(np.float32)).cuda()
    if pixel:
        up[pixel[0], 1, 1] = float(pixel[1])
    if colour:
        fr.feat[colour[0], 6:9] = float(colour[1])
    out = torch.full((sc["n"], B.FEAT_STRIDE), 7.0, dtype=torch.float32, device="cuda")
    B.render_backward(B.make_camera(c), fr, up[:3].contiguous(), up[3].contiguous(), out)
    torch.cuda.synchronize()
    return out.cpu().numpy()[:, :9]


@pytest.mark.parametrize("fillers", [0, 600])           # one batch; three, in parts where the tile is shared
@pytest.mark.parametrize("w,h", SIZES)
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_values_that_are_not_finite(value, w, h, fillers):
    sc, cam, early, late = _layers(fillers)
    base = _layer_grads(sc, cam, w, h)
    assert np.isfinite(base).all() and not base[FAINT].any()
    everywhere = early | late
    for plane in (0, 3):                                # red, transmittance
        got = _layer_grads(sc, cam, w, h, pixel=(plane, value))
        assert not got[FAINT].any()                     # composited nowhere
        np.testing.assert_allclose(got[SPOT], base[SPOT], **SAME)       # not at that pixel
        assert not np.isfinite(got[everywhere, :6]).any()
        for ch in range(3):
            if ch == plane:
                assert not np.isfinite(got[everywhere, 6 + ch]).any()
            else:
                np.testing.assert_allclose(got[everywhere, 6 + ch], base[everywhere, 6 + ch], **SAME)
    np.testing.assert_allclose(_layer_grads(sc, cam, w, h, colour=(FAINT, value)), base, **SAME)
    # the colour of an entry that is composited: it reaches what lies in front of it there, and nothing behind it
    got = _layer_grads(sc, cam, w, h, colour=(SPOT, value))
    assert not np.isfinite(got[early, :6]).any() and not np.isfinite(got[SPOT, :6]).any()
    np.testing.assert_allclose(got[early, 6:], base[early, 6:], **SAME)
    np.testing.assert_allclose(got[late], base[late], **SAME)


# ---------------------------------------------------------------- the small frames of the gradient's tests, whole tiles
@pytest.mark.parametrize("w,h,n,seed,scale_mul,opaque", [
    (37, 23, 1000, 5, 2.0, False),      # ragged tiles, pixels outside the image in the edge tiles
    (200, 120, 4000, 7, 3.0, False),    # lists of several batches
    (16, 16, 3000, 9, 1.0, False),      # one tile, a long list
    (96, 64, 2000, 13, 4.0, True),      # alpha clamped to 0.99, walks that stop early
])
def test_small_frames_in_the_corner_of_a_large_image(w, h, n, seed, scale_mul, opaque):
    """Images of up to 256 tiles share all of them.  The same frames in the last corner of an image of more than 2048
    tiles: every tile by one workgroup."""
    sc = scenes.make_scene(0, n=n, seed=seed)
    sc["scale"] = sc["scale"] * np.float32(scale_mul)
    if opaque:
        sc["opacity"] = np.where(np.arange(n) % 3 == 0, np.float32(1.0), sc["opacity"]).astype(np.float32)
    cam = dict(scenes.make_cameras(0, w, h)[0], bg=np.array([0.3, 0.1, 0.2], np.float32))
    cam = dict(cam, width=w + 1024, height=h + 512, cx=np.float32(cam["cx"] + 1024), cy=np.float32(cam["cy"] + 512))
    _compare(sc, cam, seed)
