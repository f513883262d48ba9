"""lmk_gs_preprocess_backward moves SH records and their gradients by wavefronts of 64 primitives, through LDS
where most of the 64 were binned and record by record where few were: counts around whole wavefronts and
shares of binned primitives on both sides of that line, against the oracle with the tolerance of
test_gpu_backward (per primitive 2e-4 kappa of the group's largest magnitude)."""
import numpy as np
import pytest

from paper_2503_21364_amd import scenes
from test_gpu_backward import _compare_projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n,culled", [(1, 0), (63, 0), (64, 20), (65, 30), (255, 200), (257, 100), (1000, 380)])
def test_counts_and_shares(n, culled, deg):
    sc = scenes.make_scene(0, n=n, seed=100 + n)
    sc["sh_degree"] = deg
    sc["scale"] = sc["scale"] * np.float32(2.0)
    gone = np.random.default_rng(n).permutation(n)[:culled]
    sc["mean"][2, gone] += np.float32(60.0)                 # behind the camera
    cam = scenes.make_cameras(0, 128, 96)[0]
    st = _compare_projection(sc, cam, 7 + n)
    assert st["visible"] >= n - culled - n // 4


@pytest.mark.parametrize("deg,n", [(1, 1 << 20), (2, 299_999), (2, 300_000), (2, 699_999), (2, 700_000)])
def test_both_ways_of_moving_records(deg, n):
    """From 2^20 primitives of degree 1 on, and outside 300 000 to 700 000 of degree 2, records are staged; in between the
    lanes move their own."""
    sc = scenes.make_scene(0, n=n, seed=n % 97)
    sc["sh_degree"] = deg
    gone = np.random.default_rng(n).random(n) < np.linspace(0.0, 1.0, n)       # from all binned to none
    sc["mean"][2, gone] += np.float32(60.0)
    st = _compare_projection(sc, scenes.make_cameras(0, 320, 200)[0], 3)
    assert st["visible"] > n // 3
