"""A list entry whose conic holds a NaN, or an infinity on its diagonal, reaches no pixel: the image, and the gradients of the
other entries, are those of a list without it, whichever form of the compositing kernels the tile goes by.  (Binning rule 1 keeps
no tile for such a primitive; a caller's own records, or a variance beyond fp32 under rule 0, can still hold one.)"""
import numpy as np
import pytest
import torch

from paper_2503_21364_amd import binding as B, scenes
import parity as P

pytestmark = pytest.mark.gpu

ODD = 2                                                     # the entry in question, between others


@pytest.mark.parametrize("w,h", [(16, 16), (1024, 544)])    # by cells; more than 2048 tiles, none by cells
@pytest.mark.parametrize("comp,value", [(2, np.nan), (3, np.nan), (4, np.nan), (2, np.inf), (4, np.inf)])
def test_entry_reaches_nothing(comp, value, w, h):
    cam = dict(scenes.make_camera(np.eye(3, 4), (0, 0, 0), 16, 16, 60.0, bg=(0.2, 0.4, 0.6)), width=w, height=h)
    at = lambda u, v, z: [(u - float(cam["cx"])) * z / float(cam["fx"]), (v - float(cam["cy"])) * z / float(cam["fy"]), z]
    sc = scenes.hand_placed_scene([at(8, 8, 4.0), at(3, 12, 4.5), at(7.5, 8.5, 5.0), at(9, 6, 6.0)],
                                  [(5.0,) * 3, (0.5,) * 3, (1.0,) * 3, (5.0,) * 3], opacity=[0.3, 0.6, 0.9, 0.4],
                                  sh_dc=[(0.4, 0.1, 0.2), (0.5,) * 3, (0.9, 0.8, 0.1), (0.2, 0.6, 0.3)])
    fr = P.gpu_frame(B.Scene(sc), cam, 20_000)
    assert B.read_status(fr)[1] == B.OK and int(fr.tile_offsets[1]) == 4
    rng = np.random.default_rng(1)
    rgb = np.zeros((3, h, w), np.float32)
    rgb[:, :16, :16] = rng.normal(size=(3, 16, 16))
    rgb = torch.from_numpy(rgb).cuda()

    def results():
        B.render(B.make_camera(cam), fr)
        out = torch.empty((4, B.FEAT_STRIDE), dtype=torch.float32, device="cuda")
        B.render_backward(B.make_camera(cam), fr, rgb, None, out)
        torch.cuda.synchronize()
        return fr.out_rgb.cpu().numpy(), fr.out_T.cpu().numpy(), np.delete(out.cpu().numpy(), ODD, 0)

    fr.feat[ODD, comp] = float(value)
    got = results()
    fr.feat[ODD, 5] = 0.0                                   # opacity
    fr.feat[ODD, comp] = 1.0
    want = results()
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    # the same terms, added by atomics in any order: a few 2^-24 of the sum of up to 256 terms' magnitudes
    np.testing.assert_allclose(got[2], want[2], rtol=1e-5, atol=1e-5)
