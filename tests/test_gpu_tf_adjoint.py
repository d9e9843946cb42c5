"""The adjoint with the transfer function's gradient alone: its own lanes per
ray and, for 16-bit voxels in rows of even length, loads of whole pairs of
voxels, against the FP64 oracle at the bars of test_gpu_grad.  The cameras'
rays reach every face and corner of the volume (its last row included, where a
pair would lie past the end).  The transfer function has two nodes: no sample
lies near a node, where either segment is right."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2005_01442_amd as vr  # noqa: E402
from gpu_util import DEV, log, upload_tf, upload_volume  # noqa: E402
from test_gpu_grad import REL, _check_elementwise, _rel  # noqa: E402
from test_launch_rules import field_args, rules  # noqa: E402, F401

# lanes per ray, step, image, the eye's distance over the framed one's, views
SHAPES = [(16, 0.5, 48, 1.0, 1), (4, 0.5, 200, 1.0, 1), (2, 0.5, 230, 0.35, 1), (1, 2.0, 400, 0.35, 1), (1, 2.0, 340, 1.0, 4),
          (16, 2.5, 48, 1.0, 1), (2, 2.5, 230, 0.35, 1)]
DIRECTIONS = [(-0.6, -0.65, 0.4), (0.5, 0.7, -0.6), (1.0, -0.4, 0.5), (-0.2, 0.3, 1.0)]


@pytest.mark.parametrize("nx", [42, 41])
@pytest.mark.parametrize("dtype", [np.int16, np.uint16, np.float32], ids=lambda d: d.__name__)
@pytest.mark.parametrize("group,step,size,away,views", SHAPES)
def test_tf_gradient_alone(rules, group, step, size, away, views, dtype, nx):  # noqa: F811
    dims = (nx, 26, 33)
    grid = synth.density_grid_f32(44, seed=92, smooth_sigma=2.0)[: dims[2], : dims[1], : dims[0]]
    lo, hi = (0.0, 1.0) if dtype == np.float32 else ((-1000.0, 3000.0) if dtype == np.int16 else (0.0, 60000.0))
    vol = np.ascontiguousarray(lo + (hi - lo) * grid).astype(dtype)
    tf = synth.tf_from_points([(lo, (0.1, 0.2, 0.9, 0.02)), (hi, (1.0, 0.7, 0.4, 0.3))], 2, lo, hi)
    cams = [synth.orbit_camera(dims, np.array(d), 60.0, size, size) for d in DIRECTIONS[:views]]
    centre = (np.array(dims) - 1) / 2
    for c in cams:
        c.eye = centre + away * (np.asarray(c.eye) - centre)
    assert rules.tf_adjoint_group(*field_args(dims, cams[0], views), step) == group
    g = np.random.default_rng(93).standard_normal((views, size, size, 4))
    v, t = upload_volume(vol), upload_tf(tf)
    out = vr.vr_render(v, None, cams, t, step, 0.0, False)
    _, got = vr.vr_render_backward(v, None, cams, t, step, 0.0, False, out, torch.from_numpy(g.astype(np.float32)).to(DEV),
                                   want_volume=False, want_tf=True)
    got = got.cpu().numpy().astype(np.float64)
    _, ref, _, mag = oracle.grad(vol, cams, tf, step, g, want_volume=False, magnitudes=True)
    e = _rel(got, ref)
    log(f"lanes {group} step {step} {dtype.__name__} nx {nx}: tf rel {e[0]:.2e}/{e[1]:.2e}")
    assert max(e) <= REL
    _check_elementwise(got, ref, mag, "tf", 0.99)
