// Host-side declarations shared by the lbscan translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "lbscan_device.h"

namespace lbscan {

// Arguments of one forward launch, already validated by the C entry points.
struct FwdParams {
    int batch, dim, dstate, seqlen;
    int window;
    int dtype;     // LBSCAN_FP32 / LBSCAN_BF16
    int softplus;
    int reverse;
    TokenOrder order;   // scan order of a row's tokens (kind 0: as stored)
    int pitch;          // elements from one row of a (B,D,L) or (B,N,L) tensor to the next: seqlen, or more
    const void* x;
    const void* delta;
    const void* Bm;
    const void* Cm;
    const void* z;        // nullable
    const float* A;
    const float* Dskip;   // nullable
    const float* bias;    // nullable
    const float* yprev;   // nullable, fp32 (B,D,L): added to y before the gate
    void* y;              // element type = dtype, or fp32 when y_is_f32
    int y_is_f32;         // write y as fp32 whatever dtype says (first pass of the two-pass scan)
    int force_nseg;       // >= 1: override the number of segments a row is cut into
    size_t beside;        // bytes of a first pass's result that share the scratch with the cut's summaries (0: none)
    int force_mapping;    // 0: heuristic; 1: wave-tile kernels; 2: chunk-per-lane kernel where it applies
    // Long rows are cut into nseg segments of seg_tiles forward tiles (kFwdTileTokens tokens each), one
    // block per (32 rows, segment); in_block: one per 8 rows.  carry: (nseg, N, B*D) states entering each
    // segment (read by the full pass; written by the summary pass as the states a
    // segment reaches from zero); dsum: (nseg, B*D) sum of time steps per segment.
    int nseg, seg_tiles;
    int seg_step;         // blocks from one segment to the next in the grid (set by the launcher)
    int in_block;         // full pass, at most kInBlockSegments segments: they are the waves of a block
    int summary_only;
    int fold_chain;       // full pass: fold the chain over the summaries in the kernel
    float* carry;         // nullable when nseg == 1
    float* dsum;
    // summary pass only: per-tile checkpoints for the backward pass (nullable):
    // ckpt (ntiles, B*D, N, see kCkptRows) state at the start of each tile, cum (ntiles, B*D)
    // time-step sum up to there, both counted from the start of the segment
    float* ckpt;
    float* cum;
    // summary pass for a segmented backward pass (nullable): dout (B,D,L) in, and
    // psi (nseg, N, B*D) out: the segment's summary of the right-to-left recurrence
    const void* dout;
    float* psi;
    // summary pass for window lengths that 16 is not a multiple of (nullable):
    // gck (ntiles16, N, B*D), see lbscan_fwd_wave.inc MODE 2
    float* gck;
    // forward state entering the row (nullable: zeros) and leaving it (nullable), (B*D, N)
    const float* h0;
    float* hT;
    // second pass of the path for window lengths without a compiled kernel: only
    // the local backward part, added to yprev; window is then the run-time window
    // length and the grid has one block per (32 rows, seg_tokens logical steps)
    int generic_window;
    int seg_tokens;
};

// Arguments of one backward launch: the forward inputs plus the gradient tensors.
struct BwdParams {
    int batch, dim, dstate, seqlen;
    int window;
    int dtype;
    int softplus;
    int reverse;
    TokenOrder order;
    int pitch;            // as in FwdParams; dBpart is dense
    const void* x;
    const void* delta;
    const void* Bm;
    const void* Cm;
    const void* z;        // nullable
    const float* A;
    const float* Dskip;   // nullable
    const float* bias;    // nullable
    const void* dout;
    void* dx;
    void* ddelta;
    void* dz;             // nullable iff z is
    float* dBpart;        // fp32 partial sums [dBm | dCm][block of 64 channels][B][N][L]: every
                          // block of the backward kernel writes its own share
    float* dA;            // (D,N) zeroed
    float* dDskip;        // (D) zeroed, nullable
    float* dbias;         // (D) zeroed, nullable
    const float* ckpt;    // (ntiles, B*D, N, see kCkptRows): f at the first step of every tile, counted
                          // from the start of the tile's segment
    // rows cut into nseg segments of seg_tiles backward tiles (16 tokens each):
    int nseg, seg_tiles;
    const float* cum;     // (ntiles, B*D): time-step sum from the segment start to the tile
    const float* carry;   // (nseg, N, B*D): forward state entering each segment (null: zeros)
    const float* psi_in;  // (nseg, N, B*D): psi entering each segment from the right (null: zeros)
                          // (rows not cut: both (B*D, N), as the caller holds them)
    const float* gck;     // (ntiles, N, B*D), nullable: abar_{t-1} gamma_{t-1} entering each tile
                          // (windows that straddle tile starts)
    float* dh0;           // (B*D, N), nullable: psi leaving the row on the left
};

// Arguments of the pre-scan convolution kernels (lbscan_conv.hip).
struct ConvParams {
    int batch, dim, seqlen, width;
    int dtype, activation, reverse;
    const void* x;
    const float* weight;
    const float* bias;    // nullable
    void* y;              // forward only
    const void* dy;       // backward only
    void* dx;
    float* dweight;       // (D,K), zeroed by the launcher
    float* dbias;         // (D), nullable
    int items_per_wave;   // set by the launcher
};

#ifndef LBSCAN_BWD_TILE
#define LBSCAN_BWD_TILE 16
#endif
constexpr int kTileTokens = LBSCAN_BWD_TILE;      // tokens per tile of the backward kernel = checkpoint spacing
#ifndef LBSCAN_FWD_TILE
#define LBSCAN_FWD_TILE 32
#endif
constexpr int kFwdTileTokens = LBSCAN_FWD_TILE;   // tokens per tile of the forward kernel (32: 128 bytes of an fp32 row)

// Checkpoints of f are kept by groups of rows of a batch entry, (tile, group, n, row of the group); the
// last group of an entry holds the rows that are left.
constexpr int kCkptRows = 8;

// Segments of a row that one block takes (FwdParams::in_block).
constexpr int kInBlockSegments = 8;

// Window lengths with a compiled kernel.
inline bool window_supported(int M) { return M == 1 || M == 2 || M == 4 || M == 8 || M == 16; }

// How the wave-tile kernels load the rows of a launch.  The kernels are compiled for one way each:
// with all of them in every kernel (and the pairs of ways that meet at a row's end written out) the forward
// kernels held twice the code and up to 68 spilled scalars, and lost in every
// tile what they did not use.  MI355X, us, one kernel for all ways / one for each: 128 x 768 x 197 fp32 108.6 / 107.0,
// 64 x 384 x 197 bf16, window 8, reversed 32.0 / 30.2, 1 x 256 x 8192 29.7 / 27.9, 128 x 384 x (7 x 7) by columns
// 25.7 / 22.8.
//   aligned:  whole quads (4 bytes an element, or rows that start at even ones)
//   odd:      2-byte rows that start at odd elements every other row or, walked from their end, have an
//             odd length: the aligned words around a quad
//   gathered: token by token, in a scan order
enum class Rows { aligned, odd, gathered };
inline Rows rows_of(const TokenOrder& order, int dtype, int pitch, int seqlen, int reverse)
{
    if (order.kind != 0) return Rows::gathered;
    return dtype != 0 && (pitch % 2 != 0 || (reverse && seqlen % 2 != 0)) ? Rows::odd : Rows::aligned;
}

// Forward kernels (lbscan_fwd_wave.inc), one translation unit per storage type and way.
hipError_t launch_fwd_wave_f32(const FwdParams& p, hipStream_t stream);
hipError_t launch_fwd_wave_bf16(const FwdParams& p, hipStream_t stream);
hipError_t launch_fwd_odd_bf16(const FwdParams& p, hipStream_t stream);
hipError_t launch_fwd_gather_f32(const FwdParams& p, hipStream_t stream);
hipError_t launch_fwd_gather_bf16(const FwdParams& p, hipStream_t stream);

// Chunk-per-lane forward kernel (lbscan_fwd_chunk.hip): one wave per row, 16 tokens
// per lane, no workspace.  fwd_chunk_supported: p is within what it implements.
bool fwd_chunk_supported(const FwdParams& p);
hipError_t launch_fwd_chunk(const FwdParams& p, hipStream_t stream);

// Picks the launch shape for the sizes in p and launches the forward pass
// (several kernels when rows are cut into segments).  workspace must hold
// fwd_workspace_bytes(p) bytes when that is non-zero.
// saved (nullable): buffer of saved_state_bytes(p) bytes to fill with checkpoints for
// a backward call (ignored when that size is 0).
hipError_t launch_fwd(FwdParams p, void* workspace, float* saved, hipStream_t stream);
size_t fwd_workspace_bytes(const FwdParams& p);
// The same for a window length without a compiled kernel (p.window <= p.seqlen, any
// value): two launches, the plain forward scan and the local backward part.
hipError_t launch_fwd_generic(FwdParams p, void* workspace, hipStream_t stream);
size_t fwd_generic_workspace_bytes(const FwdParams& p);
// Bytes of the saved-state buffer, 0 when rows are cut into segments (the backward
// pass then needs its own summary pass anyway).
size_t saved_state_bytes(const FwdParams& p);

// Backward kernels (lbscan_bwd_wave.inc), likewise.
hipError_t launch_bwd_wave_f32(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_wave_bf16(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_odd_bf16(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_gather_f32(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_gather_bf16(const BwdParams& p, hipStream_t stream);
// dBm, dCm (storage type) = the partial sums of BwdParams::dBpart added over the nbx
// blocks of 64 channels; bnl = B * N * L.
hipError_t launch_reduce_f32(const float* part, void* dB, void* dC, long bnl, int nbx, hipStream_t stream);
hipError_t launch_reduce_bf16(const float* part, void* dB, void* dC, long bnl, int nbx, hipStream_t stream);
// Sets n floats to zero with a kernel (a memset node must not be recorded into
// a captured graph).
hipError_t launch_zero(float* dst, long n, hipStream_t stream);
// The same for several buffers in one launch (null or empty entries are skipped).
constexpr int kZeroMany = 5;
struct ZeroMany { float* dst[kZeroMany]; long n[kZeroMany]; };
hipError_t launch_zero_many(ZeroMany z, hipStream_t stream);

// Whole backward pass: zero the accumulators, checkpoint pass, backward kernel,
// conversion of dBm / dCm when the storage type is not fp32.  dBm / dCm are the
// caller's outputs; workspace must hold bwd_workspace_bytes(f) bytes.  f.window is
// any window length >= 1 (1, 2, 4, 8, 16 run with a compiled window structure, all
// others with run-time window masks).
// saved (nullable): checkpoints left by launch_fwd on the same inputs.
// dhT (nullable): gradient arriving at the state that leaves the row.
hipError_t launch_bwd(const FwdParams& f, BwdParams p, void* dBm, void* dCm, void* workspace,
                      const float* saved, const float* dhT, hipStream_t stream);
size_t bwd_workspace_bytes(const FwdParams& f);

// Passes over reordered copies instead of gathers, for a scan order other than the
// stored one: bytes of scratch they take (0: they do not apply to p), and the launches.
size_t fwd_reordered_workspace_bytes(const FwdParams& p);
size_t bwd_reordered_workspace_bytes(const FwdParams& f);
hipError_t launch_fwd_reordered(FwdParams p, void* workspace, float* saved, hipStream_t stream);
hipError_t launch_bwd_reordered(FwdParams f, BwdParams p, void* dBm, void* dCm, void* workspace,
                                const float* saved, const float* dhT, hipStream_t stream);

// Reordering of up to kReorderMany (rows, L) tensors in one launch (lbscan_order.hip):
// dst[i][row, t] = src[i][row, map(t)] for every entry whose src is set, L at most
// kReorderMaxTokens.  Sources and destinations do not overlap.  Rows lie src_pitch[i]
// elements apart (a multiple of 4 unless it is L) and dst_pitch in every destination.
constexpr int kReorderMany = 6;
constexpr int kReorderMaxTokens = 4096;
struct ReorderMany {
    const void* src[kReorderMany];
    void* dst[kReorderMany];
    long rows[kReorderMany];
    int src_pitch[kReorderMany];
    int dst_pitch;
    const void* gate;             // launch_reorder_gate: z of entry 0 (rows as dst[0]), nullable
    long blocks[kReorderMany];    // set by the launcher
};
hipError_t launch_reorder(const ReorderMany& m, int dtype, int L, const TokenOrder& map, hipStream_t stream);
// The same from fp32 to the storage type, times SiLU(gate) where there is one.
hipError_t launch_reorder_gate(const ReorderMany& m, int dtype, int L, const TokenOrder& map, hipStream_t stream);

// Depthwise causal convolution + SiLU along the sequence and its gradient.
hipError_t launch_conv1d_fwd(const ConvParams& p, hipStream_t stream);
hipError_t launch_conv1d_bwd(const ConvParams& p, hipStream_t stream);

// Chains the per-segment summaries into the states entering each segment
// (lbscan_carry.hip): carry[s] <- exclusive scan over s of (exp(A*dsum), carry),
// started from p.h0 (zeros when null).
hipError_t launch_carry_chain(const FwdParams& p, hipStream_t stream);
// The same and, in the same launch, the chain over psi (nseg, N, B*D) walking the segments
// right to left, started from psi_init (B*D, N), zeros when null.
hipError_t launch_carry_chains(const FwdParams& p, float* psi, const float* psi_init, hipStream_t stream);
// dst[i] = src[i] (zeros when src is null), n floats.
hipError_t launch_copy(float* dst, const float* src, long n, hipStream_t stream);

}  // namespace lbscan
