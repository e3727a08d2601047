"""The bulk encoder settles only elements that are coordinates of the unit (encode_rank_mask): the basis has
r rows, and the settlement reads the row of the element it settles. The header's function is compiled for
the CPU and compared with the lane layouts over every rank, group and lane."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "kvc_internal.h"
extern "C" uint32_t rank_mask(int side, int left, int col, int grp) { return kvc::encode_rank_mask(side, left, col, grp); }
"""


@pytest.fixture(scope="module")
def mask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rank_mask")
    (d / "m.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2609_24298_amd", "csrc"), str(d / "m.cpp"), "-o", str(d / "m.so")])
    fn = ctypes.CDLL(str(d / "m.so")).rank_mask
    fn.restype = ctypes.c_uint32
    return fn


@pytest.mark.parametrize("side", [0, 1])
def test_only_coordinates_of_the_unit(mask, side):
    for r in range(2, 129, 2):
        for mc in range((r + 15) // 16):
            for lane in range(64):
                col, grp = lane & 15, lane >> 4
                want = 0
                for nt in range(4):
                    for i in range(4):
                        c = 16 * mc + (4 * grp + i if side == 0 else col)
                        want |= (c < r) << (4 * nt + i)
                assert mask(side, r - 16 * mc, col, grp) == want, (r, mc, lane)


def test_kernel_masks_before_it_settles():
    with open(os.path.join(ROOT, "paper_2609_24298_amd", "csrc", "kvc_kernels.hip")) as f:
        body = f.read()
    body = body[body.index("void encode_tiles("):]
    flag, masked, settle = (body.index(t) for t in ("ambm |= 1u", "ambm &= encode_rank_mask(side, r - 16 * mc, col, grp)",
                                                    "__ballot(ambm"))
    assert flag < masked < settle
