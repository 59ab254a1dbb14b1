"""The memory rule of the batched M2L (csrc/m2l_forms.h), compiled for the host: the float64 form's buffers are bounded
by sizes alone, and a form whose buffers cannot be had gives way to the one that needs less."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1106_5273_amd", "csrc")

SRC = r"""
#include "m2l_forms.h"
#include <stdexcept>
using namespace vfmm;
struct E { int st; };
// fails[k]: 0 fits, -2 out of memory, else another error.  Returns the form, or 100 - the error that got out;
// dropped: how often buffers were given back
extern "C" int form(int n, int required, const int *fails, int *dropped) {
    *dropped = 0;
    try {
        return first_form_that_fits<E>(n, required != 0, [&](int k) { if (fails[k]) throw E{fails[k]}; },
                                       [&] { ++*dropped; }, [](const E &e) { return e.st == -2; });
    } catch (const E &e) {
        return 100 - e.st;
    }
}
extern "C" uint64_t bytes(int rows, int pad, int64_t cells, int64_t blocks, int64_t keys, int64_t groups) {
    return f64_block_bytes(rows, pad, 24, cells, blocks, keys, groups);
}
extern "C" uint64_t most() { return MAX_F64_BYTES; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("m2l_forms")
    src, so = str(d / "wrap.cpp"), str(d / "wrap.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so])
    lib = ctypes.CDLL(so)
    lib.bytes.restype = lib.most.restype = ctypes.c_uint64
    lib.bytes.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 4
    return lib


@pytest.mark.parametrize("required,fails,want,drops", [
    (1, [0, 0], 0, 0), (1, [-2, 0], 1, 1), (1, [-2, -2], 102, 2), (1, [-6, 0], 106, 1),  # float32: two forms
    (0, [0], 0, 0), (0, [-2], 1, 1), (0, [-6], 106, 1),                                  # float64: one, or none
])
def test_form_that_fits(lib, required, fails, want, drops):
    dropped = ctypes.c_int()
    f = (ctypes.c_int * len(fails))(*fails)
    assert lib.form(len(fails), required, f, ctypes.byref(dropped)) == want
    assert dropped.value == drops


# p = 10: rows 121, padded 128; a lattice of m^3 particles in leaves of 64: (m / 4)^3 8 / 7 cells, blocks of 64 of them
# with some 189 groups each
@pytest.mark.parametrize("m,fits", [(64, True), (128, True), (256, True), (512, False), (640, False)])
def test_float64_bytes(lib, m, fits):
    cells = (m // 4) ** 3 * 8 // 7
    blocks = cells // 64
    b = lib.bytes(121, 128, cells, blocks, 1400, 189 * blocks)
    partial = 24 * 121 * 64 * (189 * blocks // 24)
    assert b >= partial and (b <= lib.most()) == fits


def test_float64_bytes_do_not_wrap(lib):
    assert lib.bytes(121, 128, 2 ** 31, 2 ** 25, 2 ** 30, 2 ** 31) >= 16 * 2 ** 55
