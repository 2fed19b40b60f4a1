"""Which contexts take their steps in one launch: the rule on the systems'
sizes, compiled for the CPU, on both sides of each of its lines."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1007_3458_amd", "csrc")


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("route")
    src, lib = d / "route.cpp", d / "route.so"
    src.write_text('#include "qsym_route.hpp"\n'
                   'extern "C" int route(const long long *off, int nsys, int cus)\n'
                   '{ return qsym::small_route(off, nsys, cus); }\n')
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", str(lib),
                           str(src)])
    L = ctypes.CDLL(str(lib))

    def call(sizes, cus=256):
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        return bool(L.route(off.ctypes.data_as(ctypes.c_void_p), len(sizes), cus))
    return call


@pytest.mark.parametrize("sizes,want", [
    ([1], True), ([192], True), ([193], False), ([256], False), ([257], False),
    ([192] * 39, True), ([200] * 4, False), ([200] * 5, True), ([225] * 20, False), ([225] * 21, True),
    ([256] * 44, False), ([256] * 45, True),
    # one large system among tiny ones: the work decides, not how many there are
    ([256] + [4] * 15, False), ([256] + [4] * 63, False), ([0, 256, 0] + [100] * 60, False),
    ([256] + [100] * 100, True), ([256] * 60 + [257], False), ([256] * 60 + [4] * 15, True),
    ([4] * 1536, True), ([4] * 1537, False), ([32] * 1537, False), ([33] * 1537, True),
    ([0] * 5000, False), ([0] * 16, True), ([192] * 4096, True)])
def test_lines_of_the_rule(route, sizes, want):
    assert route(sizes) == want


def test_rounds_follow_the_device(route):
    assert route([4] * 384, 64) and not route([4] * 385, 64)
