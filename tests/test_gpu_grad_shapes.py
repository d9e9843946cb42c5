"""The adjoint's group shapes and its box, over steps of 0.9 to 12: rays of one and
of several views, framed and close, with steps that leave the box (their taps go to
global memory), and the largest transfer function next to the box, against the FP64
oracle at the bars of test_gpu_grad.  The transfer functions are linear over more
than the value range: no sample lies at a kink (nor at the clamp of the first node,
where nearly half of these voxels, the air, would be)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import synth  # noqa: E402
from gpu_util import log  # noqa: E402
from test_gpu_grad import REL, _check_elementwise, _gpu_grad, _rel  # noqa: E402
from test_launch_rules import SCATTER, field_args, rules  # noqa: E402, F401

DIMS = (41, 26, 33)
DIRECTIONS = [(-0.6, -0.65, 0.4), (0.5, 0.7, -0.6), (1.0, -0.4, 0.5), (-0.2, 0.3, 1.0)]


# shape, views, image, the eye's distance over the framed one's, step, nodes
@pytest.mark.parametrize("shape,views,size,away,step,nodes", [
    ("4x2", 2, 330, 1.0, 0.9, 2),
    ("4x4", 4, 330, 1.0, 1.7, 2),
    ("4x4", 4, 330, 1.0, 7.0, 2),
    ("2x2", 1, 100, 1.0, 4.0, 2),
    ("box", 2, 330, 1.0, 1.7, 2),
    ("box", 1, 230, 1.0, 3.5, 2),
    ("box", 4, 330, 1.0, 5.5, 2),
    ("box", 1, 230, 0.35, 2.0, 2),
    ("box", 1, 230, 0.35, 12.0, 2),
    ("box", 1, 230, 1.0, 2.0, 1024),
])
@pytest.mark.parametrize("dtype", [np.int16, np.float32], ids=lambda d: d.__name__)
def test_gradient_shapes(rules, shape, views, size, away, step, nodes, dtype):  # noqa: F811
    grid = synth.density_grid_f32(44, seed=94, smooth_sigma=2.0)[: DIMS[2], : DIMS[1], : DIMS[0]]
    lo, hi = (0.0, 1.0) if dtype == np.float32 else (-1000.0, 3000.0)
    vol = np.ascontiguousarray(lo + (hi - lo) * grid).astype(dtype)
    lo, hi = lo - 0.02 * (hi - lo), hi + 0.02 * (hi - lo)
    tf = synth.tf_from_points([(lo, (0.1, 0.2, 0.9, 0.02)), (hi, (1.0, 0.7, 0.4, 0.3))], nodes, lo, hi)
    cams = [synth.orbit_camera(DIMS, np.array(d), 60.0, size, size) for d in DIRECTIONS[:views]]
    centre = (np.array(DIMS) - 1) / 2
    for c in cams:
        c.eye = centre + away * (np.asarray(c.eye) - centre)
    assert SCATTER[rules.adjoint_shape(*field_args(DIMS, cams[0], views), step)] == shape
    g = np.random.default_rng(95).standard_normal((views, size, size, 4))
    gv, gtf, _ = _gpu_grad(vol, tf, cams, g, step)
    rv, rt, mv, mt = oracle.grad(vol, cams, tf, step, g, magnitudes=True)
    ev, et = _rel(gv, rv), _rel(gtf, rt)
    log(f"{shape} step {step} {dtype.__name__}: grid rel {ev[0]:.2e}/{ev[1]:.2e}  tf rel {et[0]:.2e}/{et[1]:.2e}")
    assert max(ev) <= REL and max(et) <= REL
    _check_elementwise(gv, rv, mv, "grid", 0.99)
    if nodes == 2:
        _check_elementwise(gtf, rt, mt, "tf", 0.99)
