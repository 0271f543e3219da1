"""The address arithmetic of the pre-scan convolution's loads, over whole tensors on the
CPU: every load lies inside its tensor and brings every token of its quad."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_15976_amd", "csrc")

HARNESS = r"""
#include "lbscan_conv_plan.h"
using namespace lbscan;
// 0: all loads of a (rows, L) tensor of 4-byte aligned base are good; else what failed
extern "C" int check_loads(int two_byte, long rows, int L)
{
    const ConvLoads how = conv_loads(two_byte, rows, L);
    const long e = two_byte ? 2 : 4, end = rows * L * e;
    for (long r = 0; r < rows; ++r)
        for (int t0 = -4; t0 <= L + 256; t0 += 4) {
            // checked index by index in the kernel
            if (how == kLoadElements || (how == kLoadUnaligned && r == rows - 1)) continue;
            const long at = r * L + conv_quad_at(L, t0);
            const long lo = how == kLoadUnaligned ? at * e & ~3L : at * e;
            const long hi = how == kLoadUnaligned ? lo + 12 : lo + 4 * e;
            if (lo < 0 || hi > end) return 1;               // outside the tensor
            if (lo % 4) return 2;                           // not a dword address
            if (at * e < lo || (at + 4) * e > hi) return 3;
            for (int t = t0 < 0 ? 0 : t0; t < t0 + 4 && t < L; ++t)
                if (r * L + t < at || r * L + t >= at + 4) return 4;
        }
    return 0;
}
// the items that waves of `per` items hand to the element way are those of the last row
extern "C" int check_last_row(int batch, int dim, int chunks, int per)
{
    const int items = batch * chunks;
    for (int d = 0; d < dim; ++d)
        for (int i0 = 0; i0 < items; i0 += per) {
            const int n = i0 + per <= items ? per : items - i0;
            const int tail = conv_last_row_items(d, dim, i0, n, items, chunks);
            if (tail < 0 || tail > n) return 1;
            for (int i = 0; i < n; ++i) {
                const bool last = d == dim - 1 && (i0 + i) / chunks == batch - 1;
                if (last != (i >= n - tail)) return 2;
            }
        }
    return 0;
}
extern "C" int way(int two_byte, long rows, int L) { return conv_loads(two_byte, rows, L); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)], check=True)
    so = ctypes.CDLL(str(lib))
    so.check_loads.argtypes = so.way.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_int]
    return so


@pytest.mark.parametrize("two_byte", [0, 1])
def test_loads_stay_inside_the_tensor(plan, two_byte):
    for L in list(range(1, 20)) + [196, 197, 252, 253, 255, 256, 257, 505, 1025]:
        for rows in (1, 2, 3, 5):
            assert plan.check_loads(two_byte, rows, L) == 0, (L, rows)


def test_last_row_items(plan):
    plan.check_last_row.argtypes = [ctypes.c_int] * 4
    for batch in (1, 2, 5):
        for chunks in (1, 2, 7):
            for per in (1, 2, 3, 4, 8, 64):
                assert plan.check_last_row(batch, 3, chunks, per) == 0, (batch, chunks, per)


def test_ways_of_loading(plan):
    quads, unaligned, elements = 0, 1, 2
    assert [plan.way(1, 2, L) for L in (3, 4, 5, 196, 197)] == [elements, quads, unaligned, quads, unaligned]
    assert [plan.way(0, 1, L) for L in (3, 4, 5, 197)] == [elements, quads, quads, quads]
    assert plan.way(1, 1, 197) == elements                  # a single odd row: nothing after it to reach into
