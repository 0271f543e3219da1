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
extern "C" int per_wave(int bwd, long dim, long items) { return conv_items_per_wave(bwd, dim, items); }
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


def test_items_per_wave(plan):
    """Backward: one or two groups of four, whatever the type and the filter width, and few
    enough sums per channel; small calls one item per wave until the chip is full."""
    plan.per_wave.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long]
    for (B, D, chunks), want in {(1, 64, 1): 1, (24, 768, 1): 3, (48, 768, 1): 4, (56, 768, 1): 4, (72, 768, 1): 8,
                                 (80, 768, 1): 8, (128, 768, 1): 8, (512, 768, 1): 8, (96, 384, 1): 4,
                                 (16, 384, 5): 4, (1, 512, 1041): 20, (256, 768, 5): 20, (4096, 768, 4): 64}.items():
        assert plan.per_wave(1, D, B * chunks) == want, (B, D, chunks)
    for dim in (1, 3, 64, 768):
        for items in list(range(1, 300)) + [4096, 5000, 1 << 20]:
            n = plan.per_wave(1, dim, items)
            assert 1 <= n <= 64 and (n <= 4 or n % 4 == 0)
            if dim * items > 4 * 6144:
                assert n == 64 or -(-items // n) <= 64
