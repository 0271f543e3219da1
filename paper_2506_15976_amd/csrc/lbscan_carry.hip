// Carry chain of the segmented forward pass.
//
// When a row is cut into segments that different blocks scan at the same time,
// a first launch leaves, per segment s, row and state n, the state e_s the
// segment reaches from a zero state, and the sum S_s of its time steps.  The
// recurrence of Eq. 1 (Sec. 3.1) is linear, so the state entering segment s+1
// is  c_{s+1} = exp(A S_s) c_s + e_s  with c_0 = 0: the product of the
// segment's abar factors is exp(A * sum of dt).  A step of that chain is the
// affine map c -> P c + e, and affine maps compose associatively.  The summaries lie as
// (segment, n, row): a lane takes one row, so that a wave reads 256 contiguous bytes, and
// the segments of a (64 rows, n) block are shared out to its waves, kPerWave consecutive
// ones each, all loaded at once.  The waves' compositions meet in LDS, every wave folds
// those before its own, and walks its segments again from the state that enters them,
// overwriting e_s by c_s.  Chains longer than a block are walked block by block with the
// carried state passed along.  The backward pass's right-to-left recurrence
// psi_t = abar_t (e_t + psi_{t+1}) chains the same way with the segments walked from the
// last to the first, in the same launch (blockIdx.y).
// Bound by the latency of a trip to memory and of its stores.  MI355X, with a lane per segment before (every lane
// touched a line of its own) against now: forward call, 1 x 256 x 65536 (234 segments) 152 -> 146 us, 1 x 256 x
// 8192 35 -> 31; training step, which chains twice more, 563 -> 543.  A and the entering state in
// flight with the first segments' loads instead of waited for one by one before them, and the
// segments' addresses as scalar steps (3.9 instead of 5.6 KB of code, fetched anew by every launch
// between larger kernels): 1 x 192 x 8624, 5.7 -> 4.9, the forward call of 1 x 256 x 8192 30.3 -> 29.8.
// Reading several waves' compositions from LDS at once made it slower (more code).
#include "lbscan_device.h"
#include "lbscan_internal.h"

namespace lbscan {
namespace {

constexpr int kPerWave = 16;          // segments of a wave
constexpr int kChainWaves = 16;       // waves of a block, at most

// One chain: buf (nseg, N, rows) holds e_s and receives c_s; segments from the nsum-th of
// the walk on hold the identity map (their summary was not computed: nothing follows them).
struct Chain {
    float* buf;
    const float* init;                // (rows, N): the state entering the walk, nullable: zeros
    int nsum, reverse;
};
struct Chains { Chain c[2]; };

__global__ void __launch_bounds__(64 * kChainWaves)
carry_chain_kernel(const Chains chains, const float* __restrict__ dsum, const float* __restrict__ A,
                   int rows, int D, int N, int nseg)
{
    __shared__ float sP[kChainWaves][64], sE[kChainWaves][64];
    const Chain ch = chains.c[blockIdx.y];
    // (wv uniform: a segment's address is scalar work)
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int n = blockIdx.z;
    const long r0 = (long)blockIdx.x * 64 + lane;
    const bool valid = r0 < rows;
    const unsigned row = valid ? (unsigned)r0 : (unsigned)rows - 1;
    // A and the state entering the walk are loaded on every path and used behind the first
    // segments' loads, so that all of them are one trip to memory
    const float* aa = A + (long)(row % (unsigned)D) * N + n;
    float a = *aa;
    float init = *(ch.init ? ch.init + (long)row * N + n : aa);
    float cin = 0.0f;                                           // state entering the block's segments
    // from one segment of the walk to the next
    const long dstep = ch.reverse ? -(long)rows : rows, step = dstep * N;
    auto at_segment = [&](float* buf, int ss) __attribute__((always_inline)) {
        return buf + ((long)(ch.reverse ? nseg - 1 - ss : ss) * N + n) * rows;
    };
    for (int base = 0; base < nseg; base += nw * kPerWave) {
        const int first = base + wv * kPerWave;
        float P[kPerWave], e[kPerWave];
        // (segments without a summary: the last one that has one is loaded and not used)
        const int from = first < ch.nsum ? first : ch.nsum > 0 ? ch.nsum - 1 : 0;
        const float* es = at_segment(ch.buf, from);
        const float* ds = dsum + (long)(ch.reverse ? nseg - 1 - from : from) * rows;
#pragma unroll
        for (int k = 0; k < kPerWave; ++k) {
            e[k] = es[row];
            P[k] = ds[row];
            const bool more = first + k + 1 < ch.nsum;
            es += more ? step : 0;
            ds += more ? dstep : 0;
        }
        asm volatile("" : "+v"(a), "+v"(init));
        const float a2 = a * kLog2e;
        if (base == 0) cin = ch.init ? init : 0.0f;
        float Pw = 1.0f, ew = 0.0f;
#pragma unroll
        for (int k = 0; k < kPerWave; ++k) {
            const bool have = first + k < ch.nsum;
            P[k] = have ? fast_exp2(a2 * P[k]) : 1.0f;
            e[k] = have ? e[k] : 0.0f;
            ew = fmaf(P[k], ew, e[k]);
            Pw *= P[k];
        }
        sP[wv][lane] = Pw;
        sE[wv][lane] = ew;
        __syncthreads();
        float c = cin;
        for (int w = 0; w < nw; ++w) {
            if (w == wv) {
                float v = c;
                float* out = at_segment(ch.buf, first);
                if (valid) {
#pragma unroll
                    for (int k = 0; k < kPerWave; ++k) {
                        if (first + k < nseg) out[row] = v;
                        out += step;
                        v = fmaf(P[k], v, e[k]);
                    }
                }
            }
            c = fmaf(sP[w][lane], c, sE[w][lane]);
        }
        cin = c;
        __syncthreads();                  // before the compositions are overwritten
    }
}

__global__ void __launch_bounds__(256) zero_kernel(float* __restrict__ dst, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0.0f;
}

// Clears up to kZeroMany buffers in one launch: block x belongs to the buffer whose
// range of blocks contains it.
__global__ void __launch_bounds__(256) zero_many_kernel(const ZeroMany z)
{
    long blk = blockIdx.x;
#pragma unroll
    for (int k = 0; k < kZeroMany; ++k) {
        const long nb = (z.n[k] + 255) / 256;
        if (blk < nb) {
            const long i = blk * 256 + threadIdx.x;
            if (i < z.n[k]) z.dst[k][i] = 0.0f;
            return;
        }
        blk -= nb;
    }
}

__global__ void __launch_bounds__(256)
copy_kernel(float* __restrict__ dst, const float* __restrict__ src, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_chains(const FwdParams& p, const Chains& chains, int count, hipStream_t stream)
{
    const long rows = (long)p.batch * p.dim;
    const long blocks = (rows + 63) / 64 * p.dstate;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
    const int waves = (p.nseg + kPerWave - 1) / kPerWave;
    hipLaunchKernelGGL(carry_chain_kernel, dim3((unsigned)(blocks / p.dstate), count, p.dstate), dim3(64 * (waves < kChainWaves ? waves : kChainWaves)),
                       0, stream, chains, p.dsum, p.A, (int)rows, p.dim, p.dstate, p.nseg);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_zero(float* dst, long n, hipStream_t stream)
{
    if (n <= 0 || !dst) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, dst, n);
    return hipGetLastError();
}

hipError_t launch_zero_many(ZeroMany z, hipStream_t stream)
{
    long blocks = 0;
    for (int k = 0; k < kZeroMany; ++k) {
        if (!z.dst[k] || z.n[k] < 0) z.n[k] = 0;
        blocks += (z.n[k] + 255) / 256;
    }
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(zero_many_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, z);
    return hipGetLastError();
}

hipError_t launch_copy(float* dst, const float* src, long n, hipStream_t stream)
{
    if (!src) return launch_zero(dst, n, stream);
    if (n <= 0 || !dst) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_carry_chain(const FwdParams& p, hipStream_t stream)
{
    const Chains c{{{p.carry, p.h0, p.ckpt ? p.nseg : p.nseg - 1, 0}, {}}};
    return launch_chains(p, c, 1, stream);
}

hipError_t launch_carry_chains(const FwdParams& p, float* psi, const float* psi_init, hipStream_t stream)
{
    const Chains c{{{p.carry, p.h0, p.ckpt ? p.nseg : p.nseg - 1, 0}, {psi, psi_init, p.nseg, 1}}};
    return launch_chains(p, c, 2, stream);
}

}  // namespace lbscan
