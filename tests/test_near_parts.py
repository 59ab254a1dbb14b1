"""The rule that cuts the near field's lists into parts (csrc/near_parts.h), compiled for the host: every block keeps
at least one part and no more than its list has entries, and a build's targets times parts, each of which owns six
values of a buffer that 32-bit positions index, stay within the stated limit for trees of any size."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1106_5273_amd", "csrc")

SRC = r"""
#include "near_parts.h"
using namespace vfmm;
// kinds of leaves, mult[k] of each: targets, particles among them, list entries; out: per stretch tried its total
extern "C" int64_t fit(int kinds, const int64_t *mult, const int *cnt, const int *ns, const int *lc, uint64_t pairs,
                       uint64_t srcs, int64_t nent, int64_t limit, float *stretch, int64_t *most, int64_t *covered) {
    *most = 0;
    return fit_parts(limit, [&](float by) {
        const LeafWork W = leaf_work(pairs, srcs, nent, by);
        int64_t total = 0;
        *covered = 0;
        *most = 0;
        for (int k = 0; k < kinds; ++k)
            leaf_blocks(cnt[k], ns[k], [&](int, int tc, bool) {
                const int np = list_parts(W, tc, lc[k]);
                if (np < 1 || np > std::max(1, lc[k])) *covered = INT64_MIN / 2;
                total += mult[k] * np * tc;
                *covered += mult[k] * tc;
                *most = std::max<int64_t>(*most, np);
            });
        return total;
    }, *stretch);
}
extern "C" int64_t limit(int64_t n) { return partials_limit(n); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("near_parts")
    src, so = str(d / "wrap.cpp"), str(d / "wrap.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so])
    lib = ctypes.CDLL(so)
    lib.fit.restype = lib.limit.restype = ctypes.c_int64
    lib.limit.argtypes = [ctypes.c_int64]
    return lib


def _fit(lib, kinds, src_per_entry=None, limit=None):
    """kinds: (number of leaves, targets, particles, list entries)."""
    k = np.array(kinds, dtype=np.int64)
    n = int((k[:, 0] * k[:, 1]).sum())
    nent = int((k[:, 0] * k[:, 3]).sum())
    mean = src_per_entry or float((k[:, 0] * k[:, 3] * k[:, 2]).sum()) / nent
    pairs = int((k[:, 0] * k[:, 1] * k[:, 3]).sum() * mean)
    a = [np.ascontiguousarray(k[:, 0])] + [np.ascontiguousarray(k[:, j], dtype=np.int32) for j in (1, 2, 3)]
    lim = limit or lib.limit(n)
    stretch, most, covered = ctypes.c_float(), ctypes.c_int64(), ctypes.c_int64()
    tot = lib.fit(len(kinds), *[v.ctypes.data_as(ctypes.c_void_p) for v in a], ctypes.c_uint64(pairs),
                  ctypes.c_uint64(int(nent * mean)), ctypes.c_int64(nent), ctypes.c_int64(lim), ctypes.byref(stretch),
                  ctypes.byref(most), ctypes.byref(covered))
    assert covered.value == n  # every block got a part, none more than its list has entries
    assert n <= tot <= lim < 2 ** 31
    return tot, stretch.value, most.value, n


def test_limit_of_partial_results(lib):
    last = 0
    for n in (1, 1500, 2 ** 20, 2796202, 2796203, 2 ** 24, 89478485, 89478486, 2 ** 27, 2 ** 28, 4 * 10 ** 8,
              2 ** 31 - 1):
        lim = lib.limit(n)
        assert n <= lim < 2 ** 31 and lim >= last and lim >= min(4 * n, 2 ** 31 - 1)
        assert lim <= max(12 * n, 2 ** 25)
        last = lim


# 512^3 in leaves of 512: 64 parts a block times 2^27 targets is 2^33, zero in 32 bits; 448^3: wraps to a negative count
@pytest.mark.parametrize("m", [128, 256, 448, 512])
@pytest.mark.parametrize("entries", [27, 147, 1000])
def test_large_leaves_stay_within_the_limit(lib, m, entries):
    tot, stretch, most, n = _fit(lib, [((m // 8) ** 3, 512, 512, entries)])
    assert stretch >= 1.0 and most * n == tot


@pytest.mark.parametrize("kinds,src", [
    ([(2 ** 15, 64, 64, 57)], None),                      # a lattice: four parts
    ([(20000, 384, 384, 26)], None),                      # large leaves: eight parts
    ([(6000, 16, 16, 200), (3, 1, 1, 4849)], None),       # a cluster beside lone particles
    ([(1, 2 ** 31 - 1, 2 ** 31 - 1, 1)], None),           # coincident particles
    ([(2 ** 24, 20, 20, 100)], None),
    ([(10 ** 6, 130, 65, 300), (10 ** 6, 33, 0, 300)], 40.0),
    ([(4 * 10 ** 6, 100, 100, 500)], None),
])
def test_limit_and_cover(lib, kinds, src):
    tot, stretch, most, n = _fit(lib, kinds, src)
    if n <= 10 ** 7 and tot < lib.limit(n):
        assert stretch == 1.0


def test_ordinary_trees_keep_their_parts(lib):
    assert _fit(lib, [(2 ** 15, 64, 64, 57)])[1:3] == (1.0, 4)
    assert _fit(lib, [(20000, 384, 384, 26)])[1:3] == (1.0, 8)


# a limit that only one part per block meets
@pytest.mark.parametrize("cnt", [1, 33, 63, 64, 200])
def test_shortest_limit(lib, cnt):
    tot, stretch, most, n = _fit(lib, [(1000, cnt, cnt, 300)], limit=1000 * cnt)
    assert most == 1 and tot == n
