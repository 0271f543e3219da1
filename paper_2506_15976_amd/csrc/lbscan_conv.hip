// Pre-scan step of the LBMamba block (Algorithm 1: x' = SiLU(Conv1d(x))):
// depthwise causal convolution along the sequence, then SiLU, and its gradient.
//
//     pre[b,d,t] = bias[d] + sum_{k<K} w[d,k] x[b,d,t-(K-1)+k]     (inputs before 0 are zero)
//     y = pre * sigmoid(pre)          reverse: output t sees inputs t .. t+K-1 instead
//
// Both kernels are bound by HBM traffic, so the mapping serves the memory system:
// a wave takes chunks of 64 consecutive quads (256 tokens) of one row, every lane
// loads its quad once with one 16-byte load, and the K-1 neighbouring inputs an
// output needs from the quad next to it come from the neighbouring lane (a wave shift
// in the lane crossbar) instead of a second load; the quad beyond the wave's edge is
// one more load of a single sector.  A wave works on one channel and walks several
// (batch entry, chunk) items of it, so that the filter is read once, waves live
// long enough to keep loads in flight, and the backward kernel's sums over batch
// and time are folded in registers before they reach an atomic.
#include "lbscan_conv_plan.h"
#include "lbscan_device.h"
#include "lbscan_internal.h"

namespace lbscan {
namespace {

constexpr int kConvWaves = 4;          // waves per block
constexpr int kConvUnroll = 4;         // items whose loads a wave issues together

// A lane's quad x[t0 .. t0+3], zero outside the row, is fetched in two steps so that a
// wave has the loads of several items in flight: quad_issue loads without a branch (how,
// see lbscan_conv_plan.h, is a compile-time choice), quad_finish moves the elements of a
// clamped or unaligned quad into place (t0 is a multiple of four, so a quad before the row
// holds none of its tokens).
// Going back to memory for the ragged last quad and for the halo instead cost one
// memory latency each per item, on every row whose length is not a multiple of 256.
// Three more things made the compiler wait for a load before it issued the next: the 16-bit
// shift of an unaligned quad's words standing where they are loaded, the way of loading
// chosen by a run-time branch per quad, and a dword address cast from an integer (a flat
// access, waited for all at once).  With and without them (us, MI355X): forward bf16
// 64 x 384 x 197 13.0 -> 9.1, 128 x 768 x 197 44 -> 28; backward bf16 66 -> 41, fp32
// 61 -> 51 at the same shape.
struct __attribute__((packed, aligned(4))) Words2 { uint32_t v[2]; };
template <typename T> struct RawQuad;
template <> struct RawQuad<float> { Quad<float> q; };
template <> struct RawQuad<bf16_t> { Words3 w; };

template <ConvLoads HOW>
__device__ __forceinline__ RawQuad<float> quad_issue(const float* __restrict__ row, int t0, int L)
{
    if (HOW == kLoadElements) return {quad_raw_checked<float>(row, t0, t0, L)};
    return {quad_raw_fast<float>(row, conv_quad_at(L, t0))};
}
template <ConvLoads HOW>
__device__ __forceinline__ RawQuad<bf16_t> quad_issue(const bf16_t* __restrict__ row, int t0, int L)
{
    if (HOW == kLoadUnaligned) {
        const bf16_t* p = row + conv_quad_at(L, t0);
        return {*reinterpret_cast<const Words3*>(p - ((reinterpret_cast<uintptr_t>(p) >> 1) & 1))};
    }
    if (HOW == kLoadQuads) {
        const Words2 w = *reinterpret_cast<const Words2*>(row + conv_quad_at(L, t0));
        return {{{w.v[0], w.v[1], 0u}}};
    }
    const Quad<bf16_t> q = quad_raw_checked<bf16_t>(row, t0, t0, L);
    return {{{(uint32_t)q.v[0].bits | ((uint32_t)q.v[1].bits << 16),
              (uint32_t)q.v[2].bits | ((uint32_t)q.v[3].bits << 16), 0u}}};
}

template <ConvLoads HOW>
__device__ __forceinline__ Quad<float> raw_elements(const RawQuad<float>& r, const float*) { return r.q; }
template <ConvLoads HOW>
__device__ __forceinline__ Quad<bf16_t> raw_elements(const RawQuad<bf16_t>& r, const bf16_t* p)
{
    return quad_of_words(r.w, HOW == kLoadUnaligned ? p : nullptr);
}

template <typename T, ConvLoads HOW>
__device__ __forceinline__ void quad_finish(const RawQuad<T>& raw, const T* __restrict__ row, int t0, int L,
                                            float (&cur)[4])
{
    const Quad<T> q = raw_elements<HOW>(raw, row + conv_quad_at(L, t0));
#pragma unroll
    for (int e = 0; e < 4; ++e) cur[e] = to_f32(q.v[e]);
    if (HOW == kLoadElements) return;                                   // zeros are in place
    // element e is loaded element e + s; s is 0 inside the row, 1..3 for its ragged last
    // quad, anything else for a quad outside
    const int s = t0 < 0 ? 4 : (t0 > L - 4 ? t0 - (L - 4) : 0);
    const bool one = (s & 1) != 0, two = (s & 2) != 0, none = s >= 4;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = one ? (e < 3 ? cur[e < 3 ? e + 1 : 3] : 0.0f) : cur[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float w = two ? (e < 2 ? v[e < 2 ? e + 2 : 3] : 0.0f) : v[e];
        cur[e] = none ? 0.0f : w;
    }
}

// The value of the lane before (wave_shr:1) or after (wave_shl:1) this one; the lane at
// the wave's edge gets `edge`.
__device__ __forceinline__ float from_lane_before(float v, float edge)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(edge), __float_as_uint(v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float from_lane_after(float v, float edge)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(edge), __float_as_uint(v), 0x130, 0xF, 0xF, false));
}

// A value that all lanes share, kept in a vector register: a quad at a uniform position is
// otherwise moved to scalar registers as soon as it is loaded, and waited for there
// (forward bf16, 128 x 768 x 196: 31 us instead of 24).
__device__ __forceinline__ int per_lane(int v)
{
    asm("" : "+v"(v));
    return v;
}

// The lane's own quad and the three inputs on the side the filter reaches to:
// win[0..2] = x[t0-3 .. t0-1], win[3..6] = x[t0 .. t0+3] (forward direction), or
// win[0..3] = x[t0 .. t0+3], win[4..6] = x[t0+4 .. t0+6] (reversed direction).
// edge: the quad beyond the wave's first (last) one.  Every lane of the wave calls it.
template <bool REV>
__device__ __forceinline__ void make_window(const float (&cur)[4], const float (&edge)[4], float (&win)[7])
{
    if (!REV) {
#pragma unroll
        for (int j = 0; j < 3; ++j) win[j] = from_lane_before(cur[1 + j], edge[1 + j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) win[3 + e] = cur[e];
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) win[e] = cur[e];
#pragma unroll
        for (int j = 0; j < 3; ++j) win[4 + j] = from_lane_after(cur[j], edge[j]);
    }
}

// Four outputs of a row: one store where the quad lies inside the row.
template <typename T, ConvLoads HOW>
__device__ __forceinline__ void conv_store(T* __restrict__ row, int t0, int L, const float (&v)[4])
{
    if (HOW == kLoadUnaligned && t0 + 4 <= L) { quad_store_unaligned(row + t0, v); return; }
    quad_store<T>(row, t0, HOW == kLoadQuads && t0 + 4 <= L, t0, L, v);
}

// pre-activation of output e of the quad from the window above
template <int K, bool REV>
__device__ __forceinline__ float conv_at(const float (&win)[7], const float (&w)[K], float bias, int e)
{
    float pre = bias;
#pragma unroll
    for (int k = 0; k < K; ++k)
        pre = fmaf(w[k], REV ? win[e + (K - 1) - k] : win[3 + e - (K - 1) + k], pre);
    return pre;
}

// The (batch entry, chunk) items of a channel are numbered b * chunks + chunk; wave
// `wid` takes channel wid % D and the items [g * per_wave, (g + 1) * per_wave) of
// group g = wid / D, so that waves launched together work on neighbouring rows.
// Item counts fit 32 bits (checked by the launcher).
struct ConvWave {
    bool any;      // the wave has work
    int d;         // channel
    int n;         // items
    int n_last;    // how many of them, at the end, lie in the tensor's last row
    int b, ch;     // first item: batch entry and chunk
};
__device__ __forceinline__ ConvWave conv_wave(const ConvParams& p, int chunks)
{
    const unsigned items = (unsigned)p.batch * (unsigned)chunks;
    const unsigned per = (unsigned)p.items_per_wave;
    const unsigned groups = (items + per - 1) / per;
    const unsigned wid = blockIdx.x * kConvWaves + (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ConvWave w;
    w.any = wid < (unsigned)p.dim * groups;
    w.d = (int)(wid % (unsigned)p.dim);
    const unsigned i0 = (wid / (unsigned)p.dim) * per;
    w.n = (int)(i0 + per <= items ? per : items - i0);
    w.n_last = conv_last_row_items(w.d, p.dim, i0, w.n, items, chunks);
    w.b = (int)(i0 / (unsigned)chunks);
    w.ch = (int)(i0 % (unsigned)chunks);
    return w;
}

// n items of channel d, U at a time, from item (b, ch) on, which moves on behind them
template <typename T, int K, bool REV, ConvLoads HOW, int U>
__device__ __forceinline__ void conv_fwd_items(const ConvParams& p, int d, int chunks, int n, const float (&w)[K],
                                               float bias, int& b, int& ch)
{
    const int lane = threadIdx.x & 63;
    const int L = p.seqlen;
    const bool act = p.activation != 0;
    const T* __restrict__ xg = static_cast<const T*>(p.x);
    T* __restrict__ yg = static_cast<T*>(p.y);

    for (int i = 0; i < n; i += U) {
        long roff[U];
        int t0[U], th[U];                                       // th: the quad beyond the wave's edge
        RawQuad<T> raw[U], rawh[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            roff[u] = ((long)b * p.dim + d) * L;
            t0[u] = (ch * 64 + lane) * 4;
            th[u] = per_lane((ch * 64 + (REV ? 64 : -1)) * 4);
            raw[u] = quad_issue<HOW>(xg + roff[u], t0[u], L);
            rawh[u] = quad_issue<HOW>(xg + roff[u], th[u], L);
            if (i + u + 1 < n) {                                // uniform; else repeat the last item
                if (++ch == chunks) { ch = 0; ++b; }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u < n) {                                    // uniform
                float cur[4], edge[4], win[7];
                quad_finish<T, HOW>(raw[u], xg + roff[u], t0[u], L, cur);
                quad_finish<T, HOW>(rawh[u], xg + roff[u], th[u], L, edge);
                make_window<REV>(cur, edge, win);
                if (t0[u] < L) {
                    float out[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float pre = conv_at<K, REV>(win, w, bias, e);
                        out[e] = act ? pre * sigmoid_f32(pre) : pre;
                    }
                    conv_store<T, HOW>(yg + roff[u], t0[u], L, out);
                }
            }
        }
    }
    if (n > 0 && ++ch == chunks) { ch = 0; ++b; }
}

template <typename T, int K, bool REV, ConvLoads HOW>
__global__ void __launch_bounds__(64 * kConvWaves)
conv1d_fwd_kernel(const ConvParams p)
{
    const int chunks = ((p.seqlen + 3) / 4 + 63) / 64;
    const ConvWave cw = conv_wave(p, chunks);
    if (!cw.any) return;                                        // whole wave
    const int d = cw.d;
    float w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] = p.weight[(long)d * K + k];
    const float bias = p.bias ? p.bias[d] : 0.0f;
    int b = cw.b, ch = cw.ch;
    const int tail = HOW == kLoadUnaligned ? cw.n_last : 0;
    conv_fwd_items<T, K, REV, HOW, kConvUnroll>(p, d, chunks, cw.n - tail, w, bias, b, ch);
    if (tail) conv_fwd_items<T, K, REV, kLoadElements, 1>(p, d, chunks, tail, w, bias, b, ch);
}

// Gradient.  dpre_t = dy_t * dSiLU(pre_t); an input s collects w[k] dpre_t from the
// K outputs that read it, which lie in the lane's own quad and in the quad on the
// other side than the forward halo, so dpre of the neighbouring lane is shuffled
// in.  For that, consecutive chunks of a row overlap by one quad: 63 lanes own
// their quad (write dx, add to the filter and bias sums), the 64th only supplies
// dpre.  The filter and bias sums are folded over the wave's items in registers,
// then over the wave, and added with one atomic per wave and tap.
// n items of channel d, U at a time, from item (b, ch) on, which moves on behind them
template <typename T, int K, bool REV, ConvLoads HOW, int U>
__device__ __forceinline__ void conv_bwd_items(const ConvParams& p, int d, int chunks, int n, const float (&w)[K],
                                               float bias, float (&acc)[K + 1], int& b, int& ch)
{
    const int lane = threadIdx.x & 63;
    const int L = p.seqlen;
    const bool act = p.activation != 0;
    const bool owner_lane = REV ? lane >= 1 : lane <= 62;
    const T* __restrict__ xg = static_cast<const T*>(p.x);
    const T* __restrict__ gg = static_cast<const T*>(p.dy);
    T* __restrict__ dxg = static_cast<T*>(p.dx);

    for (int i = 0; i < n; i += U) {
        long roff[U];
        int t0s[U], th[U];                                      // th: the quad beyond the wave's edge
        RawQuad<T> rawx[U], rawh[U], rawg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            roff[u] = ((long)b * p.dim + d) * L;
            t0s[u] = (ch * 63 - (REV ? 1 : 0) + lane) * 4;
            th[u] = per_lane((ch * 63 + (REV ? 63 : -1)) * 4);
            rawx[u] = quad_issue<HOW>(xg + roff[u], t0s[u], L);
            rawh[u] = quad_issue<HOW>(xg + roff[u], th[u], L);
            rawg[u] = quad_issue<HOW>(gg + roff[u], t0s[u], L);
            if (i + u + 1 < n) {                                // uniform; else repeat the last item
                if (++ch == chunks) { ch = 0; ++b; }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u < n) {                                    // uniform
                const int t0 = t0s[u];
                const bool own = owner_lane && t0 >= 0 && t0 < L;
                float cur[4], edge[4], win[7], dy[4];
                quad_finish<T, HOW>(rawx[u], xg + roff[u], t0, L, cur);
                quad_finish<T, HOW>(rawh[u], xg + roff[u], th[u], L, edge);
                make_window<REV>(cur, edge, win);
                quad_finish<T, HOW>(rawg[u], gg + roff[u], t0, L, dy);

                // dpre of the own quad (zero past the end of the row: dy is zero there)
                float dpre[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float pre = conv_at<K, REV>(win, w, bias, e);
                    float g = dy[e];
                    if (act) {
                        const float sg = sigmoid_f32(pre);
                        g *= sg * fmaf(pre, 1.0f - sg, 1.0f);
                    }
                    dpre[e] = g;
                }
                // dwin: dpre around the own quad, on the side where the outputs that read it lie
                float dwin[7];
                if (!REV) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) dwin[e] = dpre[e];
#pragma unroll
                    for (int j = 0; j < 3; ++j) dwin[4 + j] = from_lane_after(dpre[j], 0.0f);
                } else {
#pragma unroll
                    for (int j = 0; j < 3; ++j) dwin[j] = from_lane_before(dpre[1 + j], 0.0f);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dwin[3 + e] = dpre[e];
                }
                if (own) {
                    float dx[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // input t0+e is read through tap k by output t0+e+(K-1)-k (forward
                        // direction) or t0+e-(K-1)+k (reversed)
                        float sum = 0.0f;
#pragma unroll
                        for (int k = 0; k < K; ++k)
                            sum = fmaf(w[k], REV ? dwin[3 + e - (K - 1) + k] : dwin[e + (K - 1) - k], sum);
                        dx[e] = sum;
                    }
                    // the quad's share is summed by itself first: a quarter of the additions into
                    // the running sums (error of dweight against 64 bits at 128 x 768 x 197:
                    // 1.8e-7 -> 1.4e-7, same time)
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        float part = 0.0f;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            part = fmaf(dpre[e], REV ? win[e + (K - 1) - k] : win[3 + e - (K - 1) + k], part);
                        acc[k] += part;
                    }
                    acc[K] += (dpre[0] + dpre[1]) + (dpre[2] + dpre[3]);
                    conv_store<T, HOW>(dxg + roff[u], t0, L, dx);
                }
            }
        }
    }
    if (n > 0 && ++ch == chunks) { ch = 0; ++b; }
}

template <typename T, int K, bool REV, ConvLoads HOW>
__global__ void __launch_bounds__(64 * kConvWaves)
conv1d_bwd_kernel(const ConvParams p)
{
    const int lane = threadIdx.x & 63;
    const int chunks = ((p.seqlen + 3) / 4 + 62) / 63;
    const ConvWave cw = conv_wave(p, chunks);
    if (!cw.any) return;                                        // whole wave
    const int d = cw.d;
    float w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) w[k] = p.weight[(long)d * K + k];
    const float bias = p.bias ? p.bias[d] : 0.0f;

    float acc[K + 1];                                           // filter taps, then bias
#pragma unroll
    for (int k = 0; k <= K; ++k) acc[k] = 0.0f;

    int b = cw.b, ch = cw.ch;
    const int tail = HOW == kLoadUnaligned ? cw.n_last : 0;
    conv_bwd_items<T, K, REV, HOW, kConvUnroll>(p, d, chunks, cw.n - tail, w, bias, acc, b, ch);
    if (tail) conv_bwd_items<T, K, REV, kLoadElements, 1>(p, d, chunks, tail, w, bias, acc, b, ch);
#pragma unroll
    for (int k = 0; k <= K; ++k) {
#pragma unroll
        for (int s = 1; s < 64; s *= 2) acc[k] += __shfl_xor(acc[k], s, 64);
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) unsafeAtomicAdd(&p.dweight[(long)d * K + k], acc[k]);
        if (p.dbias) unsafeAtomicAdd(&p.dbias[d], acc[K]);
    }
}

template <typename T, int K, bool REV, ConvLoads HOW>
hipError_t launch_conv_krh(ConvParams p, bool bwd, hipStream_t s)
{
    const long nq = (p.seqlen + 3) / 4;
    const long chunks = bwd ? (nq + 62) / 63 : (nq + 63) / 64;
    const long items = (long)p.batch * chunks;
    if (items > 0x7fffffffL) return hipErrorInvalidConfiguration;
    p.items_per_wave = conv_items_per_wave(bwd, p.dim, items);
    const long per_wave = p.items_per_wave;
    const long waves = (long)p.dim * ((items + per_wave - 1) / per_wave);
    const long blocks = (waves + kConvWaves - 1) / kConvWaves;
    if (blocks > 0x3fffffffL) return hipErrorInvalidConfiguration;     // wave ids fit 32 bits
    if (bwd)
        hipLaunchKernelGGL((conv1d_bwd_kernel<T, K, REV, HOW>), dim3((unsigned)blocks), dim3(64 * kConvWaves), 0, s, p);
    else
        hipLaunchKernelGGL((conv1d_fwd_kernel<T, K, REV, HOW>), dim3((unsigned)blocks), dim3(64 * kConvWaves), 0, s, p);
    return hipGetLastError();
}

template <typename T, int K, bool REV>
hipError_t launch_conv_kr(const ConvParams& p, bool bwd, hipStream_t s)
{
    switch (conv_loads(sizeof(T) == 2, (long)p.batch * p.dim, p.seqlen)) {
        case kLoadQuads: return launch_conv_krh<T, K, REV, kLoadQuads>(p, bwd, s);
        case kLoadUnaligned:
            if (sizeof(T) == 2) return launch_conv_krh<T, K, REV, sizeof(T) == 2 ? kLoadUnaligned : kLoadQuads>(p, bwd, s);
            return hipErrorInvalidValue;                        // (fp32 rows are never unaligned)
        default: return launch_conv_krh<T, K, REV, kLoadElements>(p, bwd, s);
    }
}

template <typename T, int K>
hipError_t launch_conv_k(const ConvParams& p, bool bwd, hipStream_t s)
{
    return p.reverse ? launch_conv_kr<T, K, true>(p, bwd, s) : launch_conv_kr<T, K, false>(p, bwd, s);
}

template <typename T>
hipError_t launch_conv_t(const ConvParams& p, bool bwd, hipStream_t s)
{
    switch (p.width) {
        case 1: return launch_conv_k<T, 1>(p, bwd, s);
        case 2: return launch_conv_k<T, 2>(p, bwd, s);
        case 3: return launch_conv_k<T, 3>(p, bwd, s);
        case 4: return launch_conv_k<T, 4>(p, bwd, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_conv1d_fwd(const ConvParams& p, hipStream_t stream)
{
    if ((long)p.batch * p.dim * p.seqlen == 0) return hipSuccess;
    return p.dtype == 0 ? launch_conv_t<float>(p, false, stream) : launch_conv_t<bf16_t>(p, false, stream);
}

hipError_t launch_conv1d_bwd(const ConvParams& p, hipStream_t stream)
{
    const ZeroMany zero{{p.dweight, p.dbias, nullptr, nullptr, nullptr}, {(long)p.dim * p.width, p.dim, 0, 0, 0}};
    hipError_t e = launch_zero_many(zero, stream);
    if (e != hipSuccess || (long)p.batch * p.dim * p.seqlen == 0) return e;
    return p.dtype == 0 ? launch_conv_t<float>(p, true, stream) : launch_conv_t<bf16_t>(p, true, stream);
}

}  // namespace lbscan
