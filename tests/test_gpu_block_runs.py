"""Block min/max at the edges of its 8-voxel runs: every row remainder, rows
shorter than a run, rows across the 512-voxel passes, every block edge and
dtype, exactly against NumPy."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2005_01442_amd as vr  # noqa: E402
from gpu_util import upload_volume  # noqa: E402

ROWS = [1, 7, 8, 9, 15, 16, 17, 18, 31, 33, 60, 61, 62, 63, 64, 65, 127, 505, 511, 512, 513, 514, 519, 520, 1023, 1025]


def reference(vol, E):
    lo = hi = vol
    for axis in range(3):
        n = vol.shape[axis]
        starts = range(0, n, E)
        cut = [slice(max(s - 1, 0), min(s + E + 1, n - 1) + 1) for s in starts]
        take = lambda a, f: np.stack([f(a[(slice(None),) * axis + (c,)], axis=axis) for c in cut], axis=axis)  # noqa: E731
        lo, hi = take(lo, np.min), take(hi, np.max)
    return np.stack([lo, hi], axis=-1).astype(np.float32)


@pytest.mark.parametrize("dtype", [np.int16, np.uint16, np.float32], ids=lambda d: d.__name__)
@pytest.mark.parametrize("edge", [4, 8, 16, 32, 64])
def test_block_ranges(edge, dtype):
    for nx in ROWS:
        ny, nz = (edge + 5, 2 * edge + 3) if nx < 200 else (edge + 1, 7)
        rng = np.random.default_rng(nx + edge)
        if dtype == np.float32:
            vol = rng.standard_normal((nz, ny, nx)).astype(np.float32)
        else:
            info = np.iinfo(dtype)
            vol = rng.integers(info.min, info.max, (nz, ny, nx), endpoint=True).astype(dtype)
        got = vr.vr_blocks_minmax(vr.vr_build_blocks(upload_volume(vol), edge)).cpu().numpy()
        assert np.array_equal(got, reference(vol, edge)), (nx, ny, nz)


def test_block_ranges_streamed_in_z():
    """Enough rows of blocks that a workgroup takes four blocks in z."""
    rng = np.random.default_rng(3)
    vol = rng.integers(-1024, 3072, (515, 521, 27)).astype(np.int16)
    got = vr.vr_blocks_minmax(vr.vr_build_blocks(upload_volume(vol), 8)).cpu().numpy()
    assert np.array_equal(got, reference(vol, 8))
