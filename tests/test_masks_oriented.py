"""The raycast's skip box on masks turned along the ray (orient_mask,
clear_ahead) against the box grown axis by axis on the mask as stored
(grow_clear_box): the same sub-blocks for every direction, and a brute-force
check that they are clear."""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_07106_amd", "csrc")

SHIM = """
#include "mvf_masks.h"
extern "C" {
uint64_t t_orient_mask(uint64_t m, uint32_t flip) { return mvf::orient_mask(m, flip); }
void t_clear_ahead(uint64_t m, uint32_t q, uint32_t* n) { mvf::clear_ahead(m, q, n); }
void t_grow_clear_box(uint64_t cm, int* lo, int* hi, const float* dir) { mvf::grow_clear_box(cm, lo, hi, dir); }
}
"""


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="mvf_masks_")
    src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "libshim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
    L = C.CDLL(so)
    L.t_orient_mask.argtypes = [C.c_uint64, C.c_uint32]
    L.t_orient_mask.restype = C.c_uint64
    L.t_clear_ahead.argtypes = [C.c_uint64, C.c_uint32, C.POINTER(C.c_uint32)]
    L.t_grow_clear_box.argtypes = [C.c_uint64, C.POINTER(C.c_int), C.POINTER(C.c_int), C.POINTER(C.c_float)]
    return L


FLIPS = [(sx, sy, sz) for sx in (1, -1) for sy in (1, -1) for sz in (1, -1)]


def _flip(d):
    return sum(3 << (2 * a) for a in range(3) if d[a] < 0)


def test_orient_mask_moves_every_bit(lib):
    for d in FLIPS:
        f = _flip(d)
        for b in range(64):
            assert lib.t_orient_mask(1 << b, f) == 1 << (b ^ f)


@pytest.mark.parametrize("density", [0.0, 0.02, 0.1, 0.3, 0.7])
def test_clear_ahead_is_the_grown_box(lib, density):
    rng = np.random.default_rng(int(1000 * density))
    for _ in range(300):
        bits = rng.random(64) < density
        m = int(sum(1 << int(b) for b in np.nonzero(bits)[0]))
        for d in FLIPS:
            f = _flip(d)
            om = lib.t_orient_mask(m, f)
            for b in rng.integers(0, 64, 8):
                b = int(b)
                s = (b & 3, (b >> 2) & 3, b >> 4)
                n = (C.c_uint32 * 3)()
                lib.t_clear_ahead(om, b ^ f, n)
                if (m >> b) & 1:
                    assert n[0] == 0
                    continue
                lo, hi = (C.c_int * 3)(*s), (C.c_int * 3)(*s)
                lib.t_grow_clear_box(m, lo, hi, (C.c_float * 3)(*d))
                for a in range(3):
                    assert n[a] == (hi[a] - s[a] + 1 if d[a] > 0 else s[a] - lo[a] + 1)
                for z in range(lo[2], hi[2] + 1):
                    for y in range(lo[1], hi[1] + 1):
                        for x in range(lo[0], hi[0] + 1):
                            assert not (m >> (16 * z + 4 * y + x)) & 1
