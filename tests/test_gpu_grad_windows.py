"""The adjoint's gradient windows: rays along every axis both ways and across
them, pixels from a fraction of a voxel to several voxels apart (windows that
move every few steps, and groups too wide for one), stencils past every face,
against the FP64 oracle at the bars of test_gpu_grad.  The transfer function
has two nodes, one segment over the whole value range: no sample lies near a
node, where either one-sided slope is right."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import synth  # noqa: E402
from test_gpu_grad import REL, _check_elementwise, _gpu_grad, _rel  # noqa: E402

DIRECTIONS = [(1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 1), (-1, 0.6, -0.3), (0.2, -1, 0.9)]


# pixels 8, 2.4, 1.2, 0.9 and 0.6 voxels apart: with the steps, every group shape of the launch rule
@pytest.mark.parametrize("size", [10, 33, 65, 90, 130])
def test_gradient_windows(size):
    dims = (41, 26, 33)
    grid = np.ascontiguousarray(synth.density_grid_f32(44, seed=90, smooth_sigma=2.0)[: dims[2], : dims[1], : dims[0]])
    tf = synth.tf_from_points([(0.0, (0.1, 0.2, 0.9, 0.02)), (1.0, (1.0, 0.7, 0.4, 0.3))], 2, 0.0, 1.0)
    cams = [synth.orbit_camera(dims, np.array(d, np.float64), 60.0, size, size - 3) for d in DIRECTIONS]
    g = np.random.default_rng(91).standard_normal((len(cams), size - 3, size, 4))
    for step in (0.5, 0.9, 1.7):
        gv, gtf, _ = _gpu_grad(grid, tf, cams, g, step)
        rv, rt, mv, mt = oracle.grad(grid, cams, tf, step, g, magnitudes=True)
        ev, et = _rel(gv, rv), _rel(gtf, rt)
        assert max(ev) <= REL and max(et) <= REL, (step, ev, et)
        _check_elementwise(gv, rv, mv, f"{size} step {step} grid", 0.99)
        _check_elementwise(gtf, rt, mt, f"{size} step {step} tf", 0.99)
