"""The diagnostics build's records are those of the last forward launch, whichever
of the forward's kernels it ran: unlit, lit, filtered."""

import glob
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2005_01442_amd")
LIBRARY = os.path.join(PACKAGE, "libvr_timeline.so")

# images of whole super-tiles in powers of two: every item of a launch has rays
PROGRAM = """
import ctypes, sys
import numpy as np, torch
import synth
import paper_2005_01442_amd as vr
from paper_2005_01442_amd import _abi
vol = synth.ct_phantom_i16(49, 45, 42, seed=140, n_soft=5, n_bone=4)
v = vr.Volume(torch.from_numpy(vol).cuda())
t = synth.tf1()
tf = vr.TF(torch.from_numpy(t.table).cuda(), t.v0, t.v1)
light = vr.Shading(**synth.SHADE_CT)
for size, how in ((64, {}), (128, dict(shading=light)), (256, dict(filter=vr.VR_FILTER_CATMULL_ROM)), (64, {}),
                  (256, dict(filter=vr.VR_FILTER_TRILINEAR)), (128, dict(shading=light))):
    counters = torch.zeros(4, dtype=torch.int64, device="cuda")
    vr.vr_render(v, None, synth.orbit_cameras((49, 45, 42), 1, 141, 60.0, size, size), tf, 0.5, counters=counters, **how)
    buf, n = np.zeros((1 << 17, 4), np.uint64), ctypes.c_uint64(0)
    _abi.check(_abi.lib().vr_timeline_read(0, buf.ctypes.data, 1 << 17, ctypes.byref(n)))
    print(size, how, n.value, int(buf[: n.value, 3].sum()), counters.tolist(), flush=True)
    assert size * size // 64 <= n.value <= size * size // 4
    assert int(buf[: n.value, 3].sum()) == int(counters[0]) > 0
"""


def test_records_of_every_forward_kernel():
    sources = glob.glob(os.path.join(PACKAGE, "csrc", "*")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    if not os.path.exists(LIBRARY) or os.path.getmtime(LIBRARY) < max(map(os.path.getmtime, sources)):
        pytest.skip("libvr_timeline.so is not built from these sources")
    run = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, env={**os.environ, "VR_LIBRARY": LIBRARY, "PYTHONPATH": ROOT},
                         capture_output=True, text=True, timeout=110)
    assert run.returncode == 0, run.stdout + run.stderr
