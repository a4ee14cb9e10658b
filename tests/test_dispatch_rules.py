"""The rules of the dispatch that are plain host code (csrc/rules.h), compiled by the host compiler: both sides of every line,
each at a shape where the other side was measured the slower one."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2205_12268_amd import wcc

CSRC = os.path.join(os.path.dirname(os.path.abspath(wcc.__file__)), "csrc")
SHIM = """
#include "rules.h"
extern "C" int shares(const wcc_desc *d, int units, int residual) {
  return wcc::shares_units(*d, units, residual != 0);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    at = tmp_path_factory.mktemp("rules")
    src, lib = at / "shim.cpp", at / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                    "-I" + os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include"), "-o", str(lib), str(src)], check=True)
    L = C.CDLL(str(lib))
    L.shares.argtypes = [C.POINTER(wcc.Desc), C.c_int, C.c_int]
    return L


def shares(rules, B, co, H, W, levels, keep, units, residual):
    d = wcc.make_desc(B, 32, co, H, W, levels, *keep, wcc.F32, 0)
    return bool(rules.shares(C.byref(d), units, int(residual)))


# shared?, B, C, H, W, keep, strip units of a plane, skip connection
FOUR_LEVELS = [
    (False, 4, 64, 256, 512, (1, 2), 64, True), (False, 4, 64, 256, 512, (1, 1), 64, True),
    (False, 4, 64, 256, 512, (1, 3), 64, True), (False, 4, 16, 128, 128, (1, 3), 8, True),
    (False, 4, 96, 64, 64, (1, 4), 2, False), (False, 1, 256, 96, 320, (1, 4), 15, False),
    (False, 4, 96, 96, 320, (1, 6), 15, False), (False, 1, 64, 256, 512, (1, 5), 64, False),
    (True, 1, 256, 128, 128, (1, 4), 8, True), (True, 4, 16, 256, 512, (1, 4), 64, True),
    (True, 4, 96, 128, 128, (1, 8), 8, False), (True, 2, 512, 64, 64, (1, 6), 2, False),
    (True, 1, 256, 256, 512, (1, 16), 64, False),
    (True, 6, 480, 16, 16, (1, 3), 1, False), (True, 16, 256, 32, 32, (3, 10), 1, False),  # planes of half a unit
    (False, 8, 128, 32, 64, (1, 4), 1, False),
]


@pytest.mark.parametrize("case", FOUR_LEVELS, ids=lambda c: "x".join(map(str, c)))
def test_inverse_at_four_levels(rules, case):
    want, B, co, H, W, keep, units, residual = case
    assert shares(rules, B, co, H, W, 4, keep, units, residual) == want


THREE_LEVELS = [
    (True, 1, 256, 128, 128, (1, 4), 8, False), (True, 16, 512, 64, 64, (1, 8), 2, False),
    (True, 4, 96, 192, 320, (1, 4), 30, False), (False, 16, 256, 128, 128, (1, 2), 8, False),
    (False, 4, 96, 136, 1024, (1, 8), 68, False),
    (False, 4, 96, 256, 512, (1, 8), 64, False), (False, 4, 96, 256, 512, (1, 10), 64, False),  # 192 MB to be stored
    (True, 4, 96, 256, 512, (1, 16), 64, False), (True, 16, 64, 128, 128, (1, 3), 8, False),
    (True, 8, 128, 128, 128, (1, 2), 8, True), (True, 4, 16, 192, 320, (1, 1), 30, True),
    # a third kept: the same for a layer, whose rows are rounded up to whole words, as for a stage call
    (True, 2, 17, 64, 64, (1, 3), 2, False), (True, 2, 512, 128, 128, (1, 3), 8, False),
    (True, 1, 16, 8, 16, (1, 3), 1, False), (True, 16, 128, 128, 128, (1, 3), 8, True),
    (False, 4, 64, 64, 64, (1, 2), 2, True), (False, 8, 128, 192, 320, (1, 4), 30, True),
]


@pytest.mark.parametrize("case", THREE_LEVELS, ids=lambda c: "x".join(map(str, c)))
def test_inverse_at_three_levels(rules, case):
    want, B, co, H, W, keep, units, residual = case
    assert shares(rules, B, co, H, W, 3, keep, units, residual) == want


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("levels", [1, 2])
def test_inverse_of_few_levels_is_not_shared(rules, levels, residual):
    assert not shares(rules, 1, 256, 128, 128, levels, (1, 16), 8, residual)
