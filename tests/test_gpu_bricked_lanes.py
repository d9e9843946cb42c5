"""Out-of-core rendering with 16, 4 and 2 lanes per ray, for every voxel type, is
bit-identical to the in-core frame, through a pool that takes many passes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import synth  # noqa: E402
from test_gpu_bricked import _bricked, _incore  # noqa: E402
from test_launch_rules import field_args, rules  # noqa: E402, F401

DIMS = (96, 80, 72)


# lanes per ray, image, the eye's distance over the framed one's
@pytest.mark.parametrize("lanes,size,away", [(16, (90, 70), 1.0), (4, (260, 220), 1.0), (2, (301, 283), 0.35), (2, (651, 640), 1.0)])
@pytest.mark.parametrize("dtype", [np.int16, np.uint16, np.float32], ids=lambda d: d.__name__)
def test_bricked_lanes_are_bit_identical_to_incore(rules, lanes, size, away, dtype):  # noqa: F811
    vol = synth.ct_phantom_i16(*DIMS, seed=66, n_soft=6, n_bone=4)
    points = synth.TF1_POINTS
    if dtype == np.uint16:
        vol = (vol.astype(np.int32) + 1024).clip(0, 4095)
        tf = synth.tf_from_points([(v + 1024, c) for v, c in points], 256, 0.0, 4080.0)
    else:
        tf = synth.tf1()
    vol = np.ascontiguousarray(vol).astype(dtype)
    cam = synth.orbit_camera(DIMS, np.array((-0.6, -0.65, 0.4)), 60.0, *size)
    centre = (np.array(DIMS) - 1) / 2
    cam.eye = centre + away * (np.asarray(cam.eye) - centre)
    assert rules.ray_group(*field_args(DIMS, cam), 0.5, 0) == lanes
    want = _incore(vol, [cam], tf, 0.5, 0.99, 16)
    got, bv = _bricked(vol, [cam], tf, 0.5, 0.99, 16, 7)
    assert bv.stats()["passes"] > 3 and want.max() > 0
    assert np.array_equal(got, want)
