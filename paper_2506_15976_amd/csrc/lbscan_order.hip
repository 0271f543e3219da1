// Reordering of row tensors between the stored token order and the scanned one
// (TokenOrder): every row of up to kReorderMany (rows, L) tensors is permuted the same
// way in one launch.
//
// Why copies: the wave-tile kernels can gather token by token, but a wave's 64 lanes
// then touch 64 sectors with every 4-byte load and the same lines are fetched again by
// every tile of the row.  Copying first moves each tensor once more, in whole lines.
// (The two ways are compared beside launch_fwd_reordered in lbscan_dispatch.hip.)
//
// What bounds it: HBM traffic, one read and one write; 5.5 TB/s measured (four row
// tensors of 128 x 768 x 197 fp32 and Bm, Cm: 115 us).  Destinations padded to whole lines are written
// whole: with the padding left out the same launch took 139 us instead of 124.  A block takes an even number of
// whole consecutive rows, which are one contiguous piece of memory: all its loads (up
// to 32 elements a thread in quads) are in flight together, go to LDS as fp32, and are
// written out token by token, 64 neighbouring tokens of a row per wave.  A lane keeps
// its tokens' places in the LDS row in registers and walks the block's rows, so the
// index arithmetic is paid once per block and not once per element.
// The gate of a wave's next kReAhead rows is loaded while it writes the rows before (the first
// ones with the block's quads): loaded where it is used, every row waited for its gate (69 us,
// 3.4 TB/s for 128 x 768 x 197 in fp32; now 49).  Rows that the block does not have are not asked
// for: long rows come two to a block, and loads of the last one in their stead made the whole
// forward call of 8 x 768 x 4096 402 us instead of 387 in bf16, 378 instead of 360 in fp32.
#include "lbscan_device.h"
#include "lbscan_internal.h"

namespace lbscan {
namespace {

constexpr int kReThreads = 256;
constexpr int kReFloats = 32 * kReThreads;            // elements of a block's rows
constexpr int kReQuads = kReFloats / 4 / kReThreads;  // quads per thread
constexpr int kReCols = 4;                            // tokens a lane holds at a time (256 of a row per wave)
constexpr int kReWaves = kReThreads / 64;
constexpr int kReAhead = 3;                           // rows whose gate a wave has in flight

// one float of padding every 32: a column of a grid whose width is a multiple of 16
// would otherwise sit in two banks
__device__ __forceinline__ int pad_slot(int i) { return i + (i >> 5); }

// dst[row, t] = src[row, map(t)]; with GATE also times SiLU(gate[row, t])
template <typename TS, typename TD, bool GATE>
__global__ void __launch_bounds__(kReThreads)
reorder_kernel(const ReorderMany m, const int L, const int rows_per_block, const TokenOrder map)
{
    __shared__ float buf[kReFloats + kReFloats / 32];
    int which = 0;
    long block = blockIdx.x;
#pragma unroll
    for (int i = 0; i + 1 < kReorderMany; ++i)
        if (which == i && block >= m.blocks[i]) { block -= m.blocks[i]; which = i + 1; }
    const long row0 = block * rows_per_block;
    const long left = m.rows[which] - row0;
    const int nrows = left < rows_per_block ? (int)left : rows_per_block;
    const int sp = m.src_pitch[which], dp = m.dst_pitch;
    const int n = nrows * sp;                                 // <= kReFloats
    const TS* __restrict__ src = static_cast<const TS*>(m.src[which]) + row0 * sp;
    TD* __restrict__ dst = static_cast<TD*>(m.dst[which]) + row0 * dp;
    const TD* __restrict__ gate = GATE ? static_cast<const TD*>(m.gate) + row0 * dp : nullptr;

    // the block's first element is an even one (even rows per block), so quads are
    // 4-byte aligned for 2-byte types too; a last quad that is not whole is loaded
    // element by element.  What lies between padded rows is loaded with them and written with
    // some token of the row: whole lines move faster than the parts of them that are needed.
    Quad<TS> q[kReQuads];
#pragma unroll
    for (int i = 0; i < kReQuads; ++i) {
        const int k = ((int)threadIdx.x + i * kReThreads) * 4;
        if (k + 4 <= n) q[i] = quad_raw_fast<TS>(src, k);
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    TD g[GATE ? kReAhead : 1][kReCols];
    auto load_gate = [&](int t0, int r0) {
#pragma unroll
        for (int u = 0; u < kReAhead; ++u) {
            const int r = r0 + kReWaves * u;
            if (r >= nrows) break;                            // (uniform)
#pragma unroll
            for (int j = 0; j < kReCols; ++j) {
                const int t = t0 + 64 * j + lane;
                g[u][j] = gate[r * dp + (t < L ? t : L - 1)];
            }
        }
    };
    if constexpr (GATE) load_gate(0, wave);
#pragma unroll
    for (int i = 0; i < kReQuads; ++i) {
        const int k = ((int)threadIdx.x + i * kReThreads) * 4;
        if (k + 4 <= n) {
#pragma unroll
            for (int e = 0; e < 4; ++e) buf[pad_slot(k + e)] = to_f32(q[i].v[e]);
        } else {
            for (int e = k; e < n; ++e) buf[pad_slot(e)] = to_f32(src[e]);
        }
    }
    __syncthreads();

    for (int t0 = 0; t0 < dp; t0 += 64 * kReCols) {
        int from[kReCols];
#pragma unroll
        for (int j = 0; j < kReCols; ++j) {
            const int t = t0 + 64 * j + lane;
            from[j] = map(t < L ? t : L - 1);
        }
        if constexpr (GATE) { if (t0 > 0) load_gate(t0, wave); }
        for (int r0 = wave; r0 < nrows; r0 += kReWaves * kReAhead) {
            float f[kReAhead][kReCols];
            if constexpr (GATE) {
#pragma unroll
                for (int u = 0; u < kReAhead; ++u)
#pragma unroll
                    for (int j = 0; j < kReCols; ++j) f[u][j] = to_f32(g[u][j]);
                if (r0 + kReWaves * kReAhead < nrows) load_gate(t0, r0 + kReWaves * kReAhead);
            }
#pragma unroll
            for (int u = 0; u < kReAhead; ++u) {
                const int r = r0 + kReWaves * u;
                if (r >= nrows) break;
#pragma unroll
                for (int j = 0; j < kReCols; ++j) {
                    const int t = t0 + 64 * j + lane;
                    float v = buf[pad_slot(r * sp + from[j])];
                    if (GATE) v *= f[u][j] * sigmoid_f32(f[u][j]);
                    if (t < dp) dst[r * dp + t] = from_f32<TD>(v);
                }
            }
        }
    }
}

template <typename TS, typename TD, bool GATE>
hipError_t launch_reorder_t(ReorderMany m, int L, const TokenOrder& map, hipStream_t s)
{
    // few rows: fewer of them to a block, down to two, so that about four blocks a CU start
    long rows = 0, total = 0;
    int widest = L;
    for (int i = 0; i < kReorderMany; ++i) {
        rows += m.src[i] ? m.rows[i] : 0;
        if (m.src[i] && m.src_pitch[i] > widest) widest = m.src_pitch[i];
    }
    if (2 * widest > kReFloats) return hipErrorInvalidValue;
    long rpb_want = (rows / 1024) & ~1L;
    const int rpb_most = (kReFloats / widest) & ~1;           // >= 2 for rows of up to kReorderMaxTokens
    const int rpb = rpb_want < 2 ? 2 : (rpb_want < rpb_most ? (int)rpb_want : rpb_most);
    for (int i = 0; i < kReorderMany; ++i) {
        m.blocks[i] = m.src[i] ? (m.rows[i] + rpb - 1) / rpb : 0;
        total += m.blocks[i];
    }
    if (total == 0) return hipSuccess;
    if (total > 0x7fffffffL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((reorder_kernel<TS, TD, GATE>), dim3((unsigned)total), dim3(kReThreads), 0, s,
                       m, L, rpb, map);
    return hipGetLastError();
}

static_assert(2 * kReorderMaxTokens <= kReFloats, "two rows fit a block's LDS");

}  // namespace

hipError_t launch_reorder(const ReorderMany& m, int dtype, int L, const TokenOrder& map, hipStream_t stream)
{
    return dtype == 0 ? launch_reorder_t<float, float, false>(m, L, map, stream)
                      : launch_reorder_t<bf16_t, bf16_t, false>(m, L, map, stream);
}

hipError_t launch_reorder_gate(const ReorderMany& m, int dtype, int L, const TokenOrder& map, hipStream_t stream)
{
    if (dtype == 0)
        return m.gate ? launch_reorder_t<float, float, true>(m, L, map, stream)
                      : launch_reorder_t<float, float, false>(m, L, map, stream);
    return m.gate ? launch_reorder_t<float, bf16_t, true>(m, L, map, stream)
                  : launch_reorder_t<float, bf16_t, false>(m, L, map, stream);
}

}  // namespace lbscan
