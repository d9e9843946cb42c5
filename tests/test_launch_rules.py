"""The launch rules (plain host arithmetic, no GPU): every piece of a launch is
covered once, and the lines of the rules lie where the measurements put them."""

import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_01442_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", out,
                    os.path.join(ROOT, "tests", "launch_rules_driver.cpp")], check=True)
    lib = ctypes.CDLL(out)
    view = [ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_double), ctypes.c_int, ctypes.c_int, ctypes.c_int]
    lib.ray_field.argtypes = [*view, ctypes.c_int, ctypes.POINTER(ctypes.c_double)]
    lib.ray_group.argtypes = [*view, ctypes.c_int, ctypes.c_double, ctypes.c_int]
    lib.preint_group.argtypes = [*view, ctypes.c_int, ctypes.c_double]
    lib.adjoint_shape.argtypes = [*view, ctypes.c_int, ctypes.c_double]
    lib.tf_adjoint_group.argtypes = [*view, ctypes.c_int, ctypes.c_double]
    lib.serve_group.argtypes = view
    lib.lanes_within.argtypes = [ctypes.c_int, ctypes.c_int64]
    lib.serve_blocks.restype = ctypes.c_int64
    lib.serve_blocks.argtypes = [ctypes.c_int64, ctypes.c_int]
    lib.serve_part.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int)]
    return lib


@pytest.mark.parametrize("lanes", [1, 2, 4, 16])
@pytest.mark.parametrize("items", [1, 1000, 2**20 - 8, 2**20 - 7, 2**20, 2**22 - 8, 2**22, 2**23 - 8, 2**23, 2**24])
def test_lanes_leave_a_launch_its_threads(rules, items, lanes):
    """A launch has fewer than 2^32 threads: as many lanes as that allows, and
    never fewer than two for it."""
    fits = [g for g in (16, 4, 2, 1) if g <= lanes and -(-items // 8) * 8 * 256 * g < 2**32]
    got = rules.lanes_within(lanes, items)
    assert got == max([*fits, min(lanes, 2)])


@pytest.mark.parametrize("parts", [2, 4, 8, 16])
@pytest.mark.parametrize("items", [1, 7, 8, 9, 64, 100, 256])
def test_serving_parts_cover_their_items_on_every_xcd(rules, items, parts):
    """Workgroup b runs on XCD b mod 8.  With any number of lanes per ray (a
    request's working parts are those below it) every working workgroup is there
    once, and no XCD has more of them than its share of the items."""
    item, part = ctypes.c_int64(), ctypes.c_int()
    seen, loads = set(), {lanes: [0] * 8 for lanes in (2, 4, 16)}
    for b in range(rules.serve_blocks(items, parts)):
        rules.serve_part(b, parts, ctypes.byref(item), ctypes.byref(part))
        assert 0 <= part.value < parts
        if item.value < items:
            assert (item.value, part.value) not in seen
            seen.add((item.value, part.value))
            for lanes, load in loads.items():
                load[b % 8] += part.value < lanes
    assert len(seen) == items * parts
    for lanes, load in loads.items():
        assert sum(load) == items * min(lanes, parts)
        assert max(load) == -(-items // 8) * min(lanes, parts)


def camera(dims, size, view):
    """(projection, eye, forward, tan(fov / 2), half extents) of the measured views."""
    n = np.array(dims, float)
    u = np.array([-0.6635568, -0.64628677, 0.37683654])
    u /= np.linalg.norm(u)
    away, fov, eye = {"framed": (1, 60, None), "far": (3, 60, None), "farther": (20, 60, None), "farthest": (40, 60, None), "near": (0.35, 60, None), "narrow": (1, 8, None),
                      "nearer": (0.6, 60, None), "inside": (0, 60, (0.5, 0.5, 0.5)), "inside_wide": (0, 90, (0.3, 0.6, 0.4)),
                      "ortho": (1, 60, None)}[view]
    where = (n - 1) / 2 + away * np.linalg.norm(n) * u if eye is None else n * eye
    half = 0.5 * float(n.max())
    return [0 if view == "ortho" else 1, *where, *-u, math.tan(math.radians(fov) / 2), half, half]


def lanes(rules, dims, size, view, views=1, step=0.5, heavy=False):
    c = camera(dims, size, view)
    return rules.ray_group((ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c[1:]), c[0], size, size, views, step, heavy)


# microseconds of int16 frames with blocks, step 0.5, by lanes per ray
S, M, L, XL = (128, 120, 100), (256, 256, 200), (512, 512, 400), (1000, 900, 700)
FRAMES = [
    (M, 128, "framed", 1, {2: 1220, 4: 510, 16: 151}),
    (M, 256, "framed", 1, {2: 797, 4: 240, 16: 181}),
    (M, 512, "framed", 1, {2: 400, 4: 330, 16: 560}),
    (L, 1024, "framed", 1, {2: 1160, 4: 1290, 16: 2850}),
    (L, 512, "framed", 1, {2: 1940, 4: 580}),
    (S, 512, "far", 16, {2: 523, 4: 735, 16: 2380}),
    (M, 512, "far", 16, {2: 1690, 4: 1067, 16: 2560}),
    (M, 512, "far", 1, {2: 1045, 4: 333, 16: 192}),
    (S, 320, "far", 1, {2: 467, 4: 154, 16: 103}),
    (M, 512, "near", 1, {2: 875, 4: 1085}),
    (M, 512, "narrow", 1, {2: 960, 4: 1193}),
    (L, 512, "narrow", 1, {2: 1758, 4: 2202}),
    (S, 512, "near", 1, {2: 491, 4: 604}),
    (M, 200, "near", 1, {2: 430, 4: 300, 16: 480}),
    (M, 512, "inside", 1, {2: 525, 4: 652}),
    (L, 256, "inside_wide", 1, {2: 573, 4: 337, 16: 597}),
    (L, 512, "inside_wide", 1, {2: 915, 4: 1077}),
    (XL, 256, "inside_wide", 1, {2: 1743, 4: 688, 16: 1031}),
    (M, 256, "ortho", 1, {2: 364, 4: 231, 16: 390}),
    (M, 512, "nearer", 1, {2: 592, 4: 659}),
    (M, 1024, "farther", 1, {2: 1344, 16: 583}),
    (M, 1024, "farther", 8, {2: 1777, 4: 1545, 16: 3953}),
    (M, 2048, "farthest", 1, {2: 1500, 4: 1106, 16: 1948}),
    (S, 2048, "farthest", 1, {2: 935, 4: 784, 16: 1880}),
    (M, 4096, "farthest", 1, {2: 2171, 16: 7713}),
]


# the same by step: large views around p = 1, with and without blocks (times near 100: relative)
H, XXL = (426, 421, 445), (700, 760, 840)
STEPPED = [
    (M, 600, "framed", 0.5, {2: 415, 4: 390}), (M, 600, "framed", 1.0, {2: 222, 4: 239}),
    (M, 512, "framed", 0.5, {2: 507, 4: 381}),
    (H, 800, "framed", 0.5, {2: 1633, 4: 1506}), (H, 800, "framed", 1.0, {2: 565, 4: 622}),
    (H, 512, "nearer", 1.0, {2: 557, 4: 613}), (H, 700, "framed", 1.0, {2: 104, 4: 100}),
    (XXL, 1150, "framed", 0.5, {2: 7561, 4: 5463}), (XXL, 1150, "framed", 1.0, {2: 2080, 4: 1843}),
    (XXL, 700, "nearer", 0.75, {2: 3423, 4: 2641}), (XXL, 600, "ortho", 1.0, {2: 2330, 4: 1848}),
    (XXL, 1000, "nearer", 0.5, {2: 93, 4: 100}), (H, 1000, "framed", 0.75, {2: 88, 4: 100}),
]


@pytest.mark.parametrize("dims,size,view,step,times", STEPPED, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_lanes_per_ray_by_step_are_the_measured_best(rules, dims, size, view, step, times):
    assert times[lanes(rules, dims, size, view, step=step)] <= 1.05 * min(times.values())


@pytest.mark.parametrize("dims,size,view,views,times", FRAMES, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_lanes_per_ray_are_the_measured_best(rules, dims, size, view, views, times):
    assert times[lanes(rules, dims, size, view, views)] <= 1.05 * min(times.values())


def test_lanes_per_ray_over_odd_cameras(rules):
    """Every accepted camera gets 2, 4 or 16 lanes: the volume behind the eye,
    extents far beyond it, images of one pixel and of the largest size, forward
    vectors of any length (which leave the answer alone)."""
    rng = np.random.default_rng(5)
    for _ in range(2000):
        dims = rng.integers(1, 900, 3)
        W, H = (int(v) for v in rng.choice([1, 3, 64, 511, 4096, 32768], 2))
        cam = [*rng.normal(0, 600, 3), *rng.normal(0, 1, 3), 10 ** rng.uniform(-4, 4), *(10 ** rng.uniform(-3, 6, 2))]
        proj, views = int(rng.integers(0, 2)), int(rng.integers(1, 17))
        args = ((ctypes.c_int32 * 3)(*map(int, dims)), (ctypes.c_double * 9)(*cam), proj, W, H)
        out = (ctypes.c_double * 4)()
        rules.ray_field(*args, views, out)
        assert all(math.isfinite(v) and v >= 0 for v in out) and out[2] <= out[1] == views * W * H
        for step in (0.1, 0.5, 1.0, 8.0):
            for heavy in (0, 1):
                assert rules.ray_group(*args, views, step, heavy) in (2, 4, 16)
        assert rules.serve_group(*args) in (2, 4, 16)
        if proj == 1:  # the same view with a longer forward vector: the plane at distance 1 moves to 3
            longer = [*cam[:3], *(3 * v for v in cam[3:6]), 3 * cam[6], 0.0, 0.0]
            other = (ctypes.c_double * 4)()
            rules.ray_field(args[0], (ctypes.c_double * 9)(*longer), 1, W, H, views, other)
            assert np.allclose(out[:], other[:], rtol=1e-9)


# microseconds of one and of twelve requests at once, by lanes per ray
REQUESTS = [
    (M, 64, "framed", {4: 841, 16: 279}, {4: 1985, 16: 828}),
    (M, 128, "near", {4: 329, 16: 304}, {4: 1443, 16: 2546}),
    (M, 200, "framed", {4: 399, 16: 228}, {4: 1410, 16: 1910}),
    (M, 256, "near", {2: 662, 4: 451}, {2: 3684, 4: 3464}),
    (M, 400, "near", {2: 1137, 4: 755}, {2: 7058, 4: 7358}),
    (M, 400, "far", {4: 720, 16: 544}, {4: 2395, 16: 2090}),
    (M, 512, "far", {4: 778, 16: 1014}, {4: 2194, 16: 2998}),
    (M, 512, "near", {2: 990, 4: 1196}, {2: 9237, 4: 11525}),
    (M, 1024, "framed", {2: 984, 4: 1118}, {2: 9749, 4: 11518}),
]


@pytest.mark.parametrize("dims,size,view,alone,twelve", REQUESTS, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_lanes_of_requests_serve_one_and_many(rules, dims, size, view, alone, twelve):
    c = camera(dims, size, view)
    g = rules.serve_group((ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c[1:]), c[0], size, size)
    assert alone[g] * twelve[g] == min(alone[k] * twelve[k] for k in alone)


# the same with pre-integration
CELLS = [
    (L, 1024, "near", {1: 5370, 2: 5818, 4: 6654}),
    (L, 1024, "narrow", {1: 4541, 2: 4729, 4: 5373}),
    (L, 1024, "inside", {1: 2912, 2: 3057, 4: 3458}),
    (M, 1024, "ortho", {1: 1980, 2: 2116, 4: 2400}),
    (S, 700, "nearer", {1: 659, 2: 700, 4: 790}),
    (S, 400, "near", {1: 411, 2: 443, 4: 453}),
    (M, 400, "nearer", {1: 800, 2: 560, 4: 514}),
    (M, 256, "near", {1: 731, 2: 404, 4: 374}),
    (L, 256, "inside", {1: 906, 2: 472, 4: 367}),
]


@pytest.mark.parametrize("dims,size,view,times", CELLS, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_lanes_per_preintegrated_ray_are_the_measured_best(rules, dims, size, view, times):
    c = camera(dims, size, view)
    g = rules.preint_group((ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c[1:]), c[0], size, size, 1, 0.5)
    assert times[g] <= 1.05 * min(times.values())


def field_args(dims, cam, views=1):
    """A camera object as the arguments of the rules' C functions."""
    c = [*map(float, cam.eye), *map(float, cam.forward), math.tan(cam.fov_y / 2), 0.0, 0.0]
    return (ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c), 1, cam.width, cam.height, views


# the adjoint with the TF gradient alone, by step
TF_ADJOINTS = [
    (M, 128, "framed", 0.5, {2: 885, 4: 432, 16: 165}),
    (M, 256, "framed", 0.5, {2: 736, 4: 419, 16: 259}),
    (M, 400, "framed", 0.5, {2: 782, 4: 411, 16: 485}),
    (M, 512, "framed", 0.5, {2: 753, 4: 625, 16: 739}),
    (M, 256, "nearer", 0.5, {2: 666, 4: 541, 16: 574}),
    (M, 256, "near", 0.5, {2: 606, 4: 699, 16: 1000}),
    (M, 400, "inside", 0.5, {2: 890, 4: 988, 16: 1409}),
    (M, 1024, "near", 0.5, {2: 8606, 4: 9488, 16: 14880}),
    (M, 128, "ortho", 4.0, {2: 138, 4: 90, 16: 78}),
    (M, 512, "far", 4.0, {2: 159, 4: 113, 16: 154}),
    (M, 256, "near", 4.0, {2: 122, 4: 149, 16: 252}),
    (M, 512, "near", 4.0, {1: 350, 2: 412, 4: 487}),
    (M, 1024, "near", 4.0, {1: 1121, 2: 1455, 4: 1783}),
    (M, 1024, "inside", 4.0, {1: 699, 2: 893, 4: 1116}),
    (M, 2048, "farther", 0.5, {2: 1061, 4: 796, 16: 1950}),
    (S, 4096, "farthest", 0.5, {2: 1223, 4: 1947}),
]


@pytest.mark.parametrize("dims,size,view,step,times", TF_ADJOINTS, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_lanes_of_the_tf_adjoint_are_the_measured_best(rules, dims, size, view, step, times):
    c = camera(dims, size, view)
    g = rules.tf_adjoint_group((ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c[1:]), c[0], size, size, 1, step)
    assert times[g] <= 1.05 * min(times.values())


# the adjoint with the grid's gradient: 4x4, 4x2 (windows placed per step, per
# sample), 2x2 and single rays per group of lanes, one box per wavefront
SCATTER = ["4x4", "4x2", "4x2s", "2x2", "1", "box"]
D = (128, 128, 128)
ADJOINTS = [
    (M, 128, "framed", 1, 0.5, (14714, 7233, 7144, 1375, 414, 7240)),
    (M, 128, "far", 1, 1.0, (2553, 1780, 1785, 1050, 303, 1756)),
    (M, 128, "near", 1, 0.5, (7789, 3236, 2848, 852, 1371, 4386)),
    (M, 128, "inside", 1, 2.0, (409, 311, 316, 384, 2710, 371)),
    (M, 256, "framed", 1, 2.0, (4015, 2643, 1568, 404, 1007, 2495)),
    (M, 256, "near", 1, 0.5, (2266, 1292, 1320, 1786, 5579, 1994)),
    (M, 256, "near", 1, 2.0, (749, 840, 829, 1428, 9461, 698)),
    (M, 256, "near", 1, 4.0, (498, 1787, 690, 1167, 9558, 462)),
    (M, 256, "inside", 1, 1.0, (730, 813, 827, 1408, 4557, 649)),
    (M, 256, "inside", 1, 2.0, (491, 709, 713, 1248, 10212, 415)),
    (M, 256, "ortho", 1, 2.0, (849, 638, 625, 766, 2071, 753)),
    (M, 400, "framed", 1, 2.0, (977, 1357, 557, 610, 2262, 852)),
    (M, 400, "near", 1, 1.4, (1588, 2001, 1999, 3502, 12870, 2009)),
    (M, 400, "near", 1, 4.0, (995, 1963, 1544, 2691, 24571, 1044)),
    (M, 400, "inside", 1, 4.0, (802, 1247, 1244, 2201, 23089, 677)),
    (M, 400, "ortho", 1, 0.5, (2485, 1899, 1954, 2132, 6162, 2634)),
    (D, 225, "framed", 16, 2.0, (3986, 4787, 2735, 3765, 23444, 2655)),
    (D, 330, "framed", 6, 2.0, (1209, 1736, 1721, 2991, 20874, 1522)),
    (D, 400, "framed", 4, 4.0, (905, 3123, 1327, 2340, 18330, 980)),
    (S, 2048, "farthest", 1, 0.5, (math.inf, math.inf, math.inf, 1185, 1883, 1568)),
]


@pytest.mark.parametrize("dims,size,view,views,step,times", ADJOINTS, ids=lambda v: str(v) if not isinstance(v, tuple) or len(v) < 6 else "")
def test_shapes_of_the_adjoint_are_the_measured_best(rules, dims, size, view, views, step, times):
    c = camera(dims, size, view)
    g = rules.adjoint_shape((ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*c[1:]), c[0], size, size, views, step)
    assert times[g] <= 1.1 * min(times), SCATTER[g]


def test_adjoint_shapes_over_odd_cameras(rules):
    """Every accepted camera and step gets a shape and lanes that are built."""
    rng = np.random.default_rng(6)
    for _ in range(2000):
        W, H = (int(v) for v in rng.choice([1, 3, 64, 511, 4096, 32768], 2))
        cam = [*rng.normal(0, 600, 3), *rng.normal(0, 1, 3), 10 ** rng.uniform(-4, 4), *(10 ** rng.uniform(-3, 6, 2))]
        args = ((ctypes.c_int32 * 3)(*map(int, rng.integers(1, 900, 3))), (ctypes.c_double * 9)(*cam), int(rng.integers(0, 2)), W, H,
                int(rng.integers(1, 17)), 10 ** rng.uniform(-2, 2))
        assert rules.adjoint_shape(*args) in range(6) and rules.tf_adjoint_group(*args) in (1, 2, 4, 16)
