"""The lanes marching a ray (16, 4 or 2, by the number of rays and the distance
between them) change nothing: a view rendered alone equals the same view
rendered among others bit for bit, and coarse views match the oracle."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2005_01442_amd as vr  # noqa: E402
from gpu_util import compare_with_flags, gpu_render, upload_tf, upload_volume  # noqa: E402

DIMS = (49, 45, 42)


def _volume(dtype):
    vol = synth.ct_phantom_i16(*DIMS, seed=140, n_soft=5, n_bone=4)
    return vol if dtype == np.int16 else vol.astype(np.float32)


@pytest.mark.parametrize("size", [(160, 120), (180, 160)], ids=["16_and_4_lanes", "4_and_2_lanes"])
@pytest.mark.parametrize("how", ["unlit", "lit", "catmull_rom", "preclassified", "trilinear"])
def test_one_view_equals_the_same_among_sixteen(size, how):
    filt = {"catmull_rom": vr.VR_FILTER_CATMULL_ROM, "preclassified": vr.VR_FILTER_BSPLINE_PRECLASSIFIED,
            "trilinear": vr.VR_FILTER_TRILINEAR}.get(how, 0)
    light = vr.Shading(**synth.SHADE_CT) if how == "lit" else None
    cams = synth.orbit_cameras(DIMS, 16, 141, 60.0, *size)
    tf = upload_tf(synth.tf1())
    for dtype in (np.int16, np.float32):
        vol = upload_volume(_volume(dtype))
        blocks = vr.vr_build_blocks(vol, 8)
        for step, ert, skip in ((0.5, 0.99, True), (1.3, 0.0, False)):
            many = vr.vr_render(vol, blocks, cams, tf, step, ert, skip, shading=light, filter=filt)
            one = vr.vr_render(vol, blocks, cams[3:4], tf, step, ert, skip, shading=light, filter=filt)
            assert torch.equal(one[0], many[3]), (dtype, step)


@pytest.mark.parametrize("size", [7, 16, 31, 44])
def test_coarse_views_match_oracle(size):
    """Rays 2 to 14 voxels apart, ragged tiles, odd rows."""
    vol = _volume(np.int16)
    cams = synth.orbit_cameras(DIMS, 3, 142, 60.0, size + 2, size)
    ref = oracle.render(vol, cams, synth.tf1(), 0.5, ert=0.99)
    got = gpu_render(vol, cams, synth.tf1(), 0.5, 0.99, True, block_edge=8)
    compare_with_flags(got, ref["rgba"], ref["flags"], 0.99)


@pytest.mark.parametrize("size", [(160, 120), (180, 160)], ids=["16_and_4_lanes", "4_and_2_lanes"])
def test_preintegrated_view_equals_the_same_among_sixteen(size):
    cams = synth.orbit_cameras(DIMS, 16, 143, 60.0, *size)
    tf = upload_tf(synth.tf1())
    for dtype in (np.int16, np.float32):
        vol = upload_volume(_volume(dtype))
        blocks = vr.vr_build_blocks(vol, 8)
        for step, ert, skip in ((0.5, 0.99, True), (1.3, 0.0, False), (2.5, 0.9, True)):
            table = vr.vr_preint_build(tf, step)
            many = vr.vr_render_preint(vol, blocks, cams, tf, table, step, ert, skip)
            one = vr.vr_render_preint(vol, blocks, cams[5:6], tf, table, step, ert, skip)
            full = vr.vr_render_preint(vol, None, cams[5:6], tf, table, step, ert, False)
            assert torch.equal(one[0], many[5]) and torch.equal(one, full), (dtype, step)


@pytest.mark.parametrize("dtype", [np.int16, np.float32], ids=lambda d: d.__name__)
@pytest.mark.parametrize("step,ert,skip", [(0.5, 0.99, True), (1.3, 0.0, False), (2.5, 0.9, True)])
def test_close_preintegrated_view_equals_the_same_among_far_ones(dtype, step, ert, skip):
    """A view whose rays all cross takes one lane per ray; among far views (rays
    that miss) it takes two."""
    near, *far = synth.orbit_cameras(DIMS, 8, 145, 60.0, 640, 620)
    centre = (np.array(DIMS) - 1) / 2
    near.eye = centre + 0.3 * (near.eye - centre)
    for c in far:
        c.eye = centre + 4.0 * (c.eye - centre)
    vol, tf = upload_volume(_volume(dtype)), upload_tf(synth.tf1())
    blocks, table = vr.vr_build_blocks(vol, 8), vr.vr_preint_build(tf, step)
    one = vr.vr_render_preint(vol, blocks, [near], tf, table, step, ert, skip)
    many = vr.vr_render_preint(vol, blocks, [near, *far], tf, table, step, ert, skip)
    assert float(one.max()) > 0 and torch.equal(one[0], many[0])


@pytest.mark.parametrize("nodes", [2, 3, 130, 257])
@pytest.mark.parametrize("opacity", [0.0, 0.3, 60.0])
def test_preint_table_sizes(nodes, opacity):
    rng = np.random.default_rng(nodes)
    table = rng.random((nodes, 4)).astype(np.float32)
    table[:, 3] *= opacity
    table[:: 3, 3] = 0.0
    tf = synth.TransferFunction(table, -1.0, 2.0)
    for step in (0.25, 8.0):
        got = vr.vr_preint_table(vr.vr_preint_build(upload_tf(tf), step)).cpu().numpy()
        # (the bar of test_gpu_preint: both sides integrate in FP64, entries lie in [0, 1] and are stored as fp32)
        assert np.abs(got - oracle.preint_table(tf, step)).max() <= 1e-6


@pytest.mark.parametrize("size", [(40, 33), (180, 160)], ids=["16_lanes", "4_lanes"])
def test_nan_voxels_classify_as_the_first_node(size):
    """A NaN value takes the TF's first node (coordinate 0) on every lane: an
    all-NaN volume gives the image of an all-zero volume under a TF from 0, bit
    for bit (zero is reconstructed exactly)."""
    tf = synth.tf1()
    table = torch.from_numpy(np.ascontiguousarray(tf.table)).cuda()
    table[0] = torch.tensor([0.2, 0.5, 0.8, 0.07])
    tf = vr.TF(table, 0.0, 1000.0)
    cams = synth.orbit_cameras(DIMS, 1, 144, 60.0, *size)
    images = []
    for value in (np.nan, 0.0):
        vol = upload_volume(np.full(DIMS[::-1], value, np.float32))
        images.append(vr.vr_render(vol, None, cams, tf, 0.5, 0.99, False))
    assert float(images[0].max()) > 0 and torch.equal(images[0], images[1])
