"""Occupancy planes and workgroup order of a frame, made in one launch: leaping
over empty blocks changes no bit of an image, on block grids one block wide,
on rows and planes that cross words and workgroups, and for views past the
first launch (whose order is made alone)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import synth  # noqa: E402
import paper_2005_01442_amd as vr  # noqa: E402
from gpu_util import upload_volume  # noqa: E402


@pytest.mark.parametrize("dims", [(6, 6, 6), (7, 6, 150), (150, 7, 6), (61, 9, 203), (131, 133, 60)],
                         ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("blobs", [0, 1, 6])
def test_leaps_change_nothing(dims, blobs):
    rng = np.random.default_rng(160 + blobs + dims[0])
    vol = np.zeros(dims[::-1], np.int16)
    for _ in range(blobs):  # single bright voxels, at faces and corners too
        z, y, x = (int(rng.choice([0, n - 1, rng.integers(n)])) for n in vol.shape)
        vol[z, y, x] = 900
    table = np.zeros((129, 4), np.float32)
    table[3:, :3] = rng.uniform(0.1, 1.0, (126, 3))
    table[3:, 3] = 0.8
    cams = synth.orbit_cameras(dims, 18, 161, 60.0, 40, 33)
    volume, tf = upload_volume(vol), vr.TF(torch.from_numpy(table).cuda(), 0.0, 1000.0)
    for edge in (4, 8):
        blocks = vr.vr_build_blocks(volume, edge)
        full = vr.vr_render(volume, None, cams, tf, 0.5, 0.0, False)
        leap = vr.vr_render(volume, blocks, cams, tf, 0.5, 0.0, True)
        assert torch.equal(full, leap), edge
