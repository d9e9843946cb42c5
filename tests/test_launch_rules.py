"""The launch rules (plain host arithmetic, no GPU): every piece of a launch is
covered once, and the lines of the rules lie where the measurements put them."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_01442_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", out,
                    os.path.join(ROOT, "tests", "launch_rules_driver.cpp")], check=True)
    lib = ctypes.CDLL(out)
    lib.serve_blocks.restype = ctypes.c_int64
    lib.serve_blocks.argtypes = [ctypes.c_int64, ctypes.c_int]
    lib.serve_part.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int)]
    return lib


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
