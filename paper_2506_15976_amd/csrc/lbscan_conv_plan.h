// How the pre-scan convolution's kernels load the quads of a row: the address arithmetic,
// in plain C++ so that it can be checked over whole tensors on the CPU.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define LBSCAN_PLAN_FN __host__ __device__ __forceinline__
#else
#define LBSCAN_PLAN_FN inline
#endif

namespace lbscan {

// kLoadQuads      one quad (4 elements) from a position clamped into the row
// kLoadUnaligned  2-byte rows of odd length, half of which start between two dwords: the
//                 12 aligned bytes around that position.  They reach up to two elements
//                 past the quad, so the tensor's last row is loaded element by element.
// kLoadElements   rows of fewer than four tokens, and a single odd row: element by element
enum ConvLoads { kLoadQuads, kLoadUnaligned, kLoadElements };

LBSCAN_PLAN_FN ConvLoads conv_loads(bool two_byte, long rows, int L)
{
    if (L < 4) return kLoadElements;
    if (!two_byte || L % 2 == 0) return kLoadQuads;
    return rows < 2 ? kLoadElements : kLoadUnaligned;
}

// Token of a row at which the load of quad t0 (any multiple of four, also outside the row)
// starts.  Not for kLoadElements.
LBSCAN_PLAN_FN int conv_quad_at(int L, int t0) { return t0 < 0 ? 0 : (t0 > L - 4 ? L - 4 : t0); }

// How many of a wave's items, taken from the end, lie in the tensor's last row: channel d
// of dim, the items [i0, i0 + n) of the channel's `items`, `chunks` of them to a row.
LBSCAN_PLAN_FN int conv_last_row_items(int d, int dim, unsigned i0, int n, unsigned items, int chunks)
{
    const long in = (long)i0 + n - ((long)items - chunks);
    return d != dim - 1 || in <= 0 ? 0 : (in < n ? (int)in : n);
}

}  // namespace lbscan
