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

// Items ((batch entry, chunk) pairs of a channel) per wave.  Forward: about 8 waves per
// SIMD of the chip in all.  Backward: one group of the four items whose loads are in flight
// together, two groups where that still makes 8 waves per SIMD and more: shorter waves fill
// the chip's last round better than waves that fit it in one round.  Measured (fp32, K = 4,
// us, 4 / 8 / one round of 6 waves per SIMD): 48 x 768 x 197 23.2 / 24.1 / 24.1,
// 72 x 768 x 197 30.7 / 32.2 / 32.6 and 26.8 / 25.5 / 25.3 with inputs in the Infinity
// Cache, 128 x 768 x 197 48.2 / 50.5 / 51.6 and 41.5 / 41.3 / 41.4, 16 x 384 x 1025
// 21.7 / 21.2 / 22.8, 512 x 768 x 197 171 / 183 / 199; K = 1..3 and bf16 alike within 3%.
// Each wave adds its sums to the channel's with fp32 atomics: at most 64 of them meet there
// (until waves are 64 items long), or their rounding would outgrow that of longer waves.
LBSCAN_PLAN_FN int conv_items_per_wave(bool bwd, long dim, long items)
{
    const long resident = bwd ? 6 * 1024 : 8 * 1024;
    long per = (dim * items + resident - 1) / resident;
    if (bwd && per > 4) {
        const long meet = (items + 255) / 256 * 4;          // whole groups, 64 sums
        per = per < 8 ? 4 : 8;
        per = per < meet ? meet : per;
    }
    return (int)(per < 1 ? 1 : (per > 64 ? 64 : per));
}

}  // namespace lbscan
