"""Interpolating-spline prefilter at the edges of its segment split: rows of
one to sixteen voxels per lane (and past them), lines of one to sixteen
segments of 64 (and past them), every dtype, against the FP64 oracle."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2005_01442_amd as vr  # noqa: E402
from gpu_util import log, upload_volume  # noqa: E402

SHAPES_XYZ = [(1, 1, 1), (2, 3, 1), (1, 64, 65), (63, 65, 2), (64, 16, 17), (65, 129, 33), (513, 5, 3), (1024, 2, 64),
              (1025, 3, 2), (3, 1024, 2), (2, 1025, 3), (5, 2, 1023), (2, 1, 1100)]


@pytest.mark.parametrize("shape", SHAPES_XYZ, ids=str)
@pytest.mark.parametrize("dtype", [np.int16, np.uint16, np.float32], ids=lambda d: d.__name__)
def test_prefilter_segments(shape, dtype):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx * 7 + ny * 3 + nz)
    lo, hi = (0, 4096) if dtype == np.uint16 else (-1024, 3072)
    vol = rng.integers(lo, hi, (nz, ny, nx)).astype(dtype)
    ref = oracle.prefilter(vol)
    got = vr.vr_prefilter_bspline(upload_volume(vol)).tensor.cpu().numpy().astype(np.float64)
    # the inverse of one axis has norm 3, so |c| <= 27 max|v|; each axis rounds
    # a handful of times per voxel, its errors damped by 0.27 per voxel both
    # ways: under 8 eps of the largest coefficient per axis
    bound = 3 * 8 * 2.0**-24 * 27 * np.abs(vol.astype(np.float64)).max()
    d = np.abs(got - ref).max()
    log(f"prefilter {shape} {dtype.__name__}: max |d| {d:.3e} of {bound:.3e}")
    assert d <= bound


@pytest.mark.parametrize("shape", [(65, 3, 3), (700, 2, 2), (3, 300, 2), (2, 3, 200)], ids=str)
def test_infinite_voxel_reaches_its_lines(shape):
    """An infinite voxel makes every coefficient infinite, with the sign that
    alternates along each axis, as sweeps over whole lines give; no NaN."""
    nx, ny, nz = shape
    vol = np.ones((nz, ny, nx), np.float32)
    at = (nz // 2, ny // 2, nx // 3)
    vol[at] = np.inf
    got = vr.vr_prefilter_bspline(upload_volume(vol)).tensor.cpu().numpy()
    z, y, x = np.meshgrid(np.arange(nz) - at[0], np.arange(ny) - at[1], np.arange(nx) - at[2], indexing="ij")
    assert np.array_equal(got, np.where((z + y + x) % 2 == 0, np.inf, -np.inf).astype(np.float32))


@pytest.mark.parametrize("nx", [2, 3, 5, 8, 9, 16, 17, 32, 33, 64])
def test_prefilter_short_rows(nx):
    """Several rows to a wavefront: rows that fill their lanes, rows that leave
    some idle, a last workgroup that is not full."""
    rng = np.random.default_rng(nx)
    vol = rng.integers(-1024, 3072, (3, 131, nx)).astype(np.int16)
    got = vr.vr_prefilter_bspline(upload_volume(vol)).tensor.cpu().numpy().astype(np.float64)
    bound = 3 * 8 * 2.0**-24 * 27 * np.abs(vol.astype(np.float64)).max()  # as above
    assert np.abs(got - oracle.prefilter(vol)).max() <= bound


def test_prefilter_of_very_many_rows():
    """2^26 rows: a wavefront per row would be 2^32 threads, which no launch
    takes.  Volumes constant along y and z keep their row's coefficients."""
    row = torch.tensor([100, 700], dtype=torch.int16, device="cuda")
    vol = vr.Volume(row.expand(8192, 8192, 2).contiguous())
    got = vr.vr_prefilter_bspline(vol).tensor
    want = oracle.prefilter(np.array([[[100, 700]]], np.int16))[0, 0]
    d = float((got - torch.from_numpy(want).to(got)).abs().max())
    assert d <= 3 * 8 * 2.0**-24 * 27 * 700


@pytest.mark.parametrize("length", [200, 256, 512, 1000])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_prefilter_far_from_the_data_is_zero(axis, length):
    """The coefficients fall off by 2 - sqrt(3) a voxel: 120 voxels from the last
    voxel other than zero they are below the least fp32 number, zero.  A line's
    first voxels are the largest, then its last."""
    for at in (slice(0, 3), slice(length - 3, length)):
        vol = np.zeros((length, 2, 2), np.float32)
        vol[at] = 60000.0
        vol = np.ascontiguousarray(np.moveaxis(vol, 0, axis))
        got = vr.vr_prefilter_bspline(upload_volume(vol)).tensor.cpu().numpy()
        line = np.abs(np.moveaxis(got, axis, 0)).max(axis=(1, 2))
        far = line[123:] if at.start == 0 else line[: length - 123]
        assert line.max() > 60000.0 and far.max() == 0.0
