// Device-side helpers shared by the lbscan HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbscan {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// 2^v through the hardware transcendental (v_exp_f32), without the range
// fix-ups of the library exp2f: arguments here are <= ~30 and results that
// underflow may flush to zero.
__device__ __forceinline__ float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ __forceinline__ float fast_log2(float v) { return __builtin_amdgcn_logf(v); }
__device__ __forceinline__ float fast_rcp(float v) { return __builtin_amdgcn_rcpf(v); }

// softplus(v) = log(1 + exp(v)), v > 20 -> v (Algorithm 1's Delta line), and its
// derivative sigma(v) = e / (1 + e) (1 above 20).  The time step multiplies every
// state update, so it is kept to a few ulp, in one branch-free form for all v:
// with e = exp(v) and w = fl(1 + e),
//     log(1 + e) = log(w) + (e - (w - 1)) / w        (up to O(ulp^2)),
// where the second term restores the bits lost when 1 + e was rounded (it is all
// of the result for e < 2^-24).  v_log_f32 is accurate to ~1e-7 of its result
// also for arguments next to 1 (measured on MI355X: 1.1e-7 over w - 1 in
// [1e-7, 1]), so no series is needed there.  For v > 88 e overflows to inf and
// the sum becomes NaN; the selects below discard it.
__device__ __forceinline__ float softplus_f32(float v, float& dsoftplus)
{
    const float e = fast_exp2(v * kLog2e);
    const float w = 1.0f + e;
    const float rw = fast_rcp(w);
    const float r = fmaf(fast_log2(w), kLn2, (e - (w - 1.0f)) * rw);
    const bool lin = v > 20.0f;
    dsoftplus = lin ? 1.0f : e * rw;
    return lin ? v : r;
}
__device__ __forceinline__ float softplus_f32(float v)
{
    float unused;
    return softplus_f32(v, unused);
}

__device__ __forceinline__ float sigmoid_f32(float v)
{
    return fast_rcp(1.0f + fast_exp2(-v * kLog2e));
}

// ---- scan order ------------------------------------------------------------
// The order in which a row's tokens are scanned: index t of the scanned sequence ->
// index of the token as stored.  kind 0: the tokens as stored.  kind 1: the tokens
// [prefix, prefix + H W) are an H x W grid stored row by row and are scanned column
// by column, top to bottom (the vertical scans of the multi-direction models of
// Sec. 4.5 / Appendix D); tokens before and after the grid (class tokens) keep
// their places.  Set by the host; H > 0 also for kind 0.
struct TokenOrder {
    int kind, prefix, H, W, HW;
    float rH;          // 1 / H
    __device__ __forceinline__ int operator()(int t) const
    {
        if (kind == 0) return t;
        const int k = t - prefix;
        // column c = k / H: the float quotient is off by at most one for k < 2^24
        int c = (int)((float)k * rH);
        int r = k - c * H;
        const int low = r < 0, high = r >= H, off = high - low;
        const int in_grid = prefix + (r - off * H) * W + c + off;
        // (values chosen between, not ways taken: a branch here would stand before every load)
        return (unsigned)k < (unsigned)HW ? in_grid : t;
    }
};

// ---- storage types -------------------------------------------------------
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
// round to nearest even; NaN stays NaN (gfx950 converts in hardware, two values per
// v_cvt_pk_bf16_f32 where the compiler can pair them)
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v)
{
    bf16_t o;
    o.bits = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
    return o;
}

// Four consecutive elements.  Global memory on gfx950 serves multi-dword
// accesses at dword alignment, so the fp32 quad only promises 4-byte alignment
// (rows of odd length start at any dword); the bf16 quad promises 4 bytes too:
// where a row can start at an odd element callers load the words around a quad
// (Words3) and use quad_store_unaligned inside the row, and element accesses at its
// ragged end.
template <typename T> struct Quad;
template <> struct __attribute__((packed, aligned(4))) Quad<float> { float v[4]; };
template <> struct __attribute__((packed, aligned(4))) Quad<bf16_t> { bf16_t v[4]; };

// One quad of a (rows, L) tensor in its storage type, for later conversion.  `base` is
// uniform, `off` the element offset of quad element 0 and `ph` its token index.  The fast
// form is one unconditional quad load.  The checked form (further down) zeroes elements
// whose token index ph + e is outside [0, L), loading from a clamped (always valid)
// address.  Where the tokens of a scan order are gathered the loads are unconditional: a value
// chosen between structs, or an index computed in a branch, becomes a branch that the
// load is moved into, and the quad's loads wait for one another (4 x 384 x (37 x 37) by columns, bf16,
// 72.6 -> 65.1 us).  In stored order such branches stand: the ragged chunks of the chunk kernel skip
// what lies behind the row (unconditional, 1 x 192 x 900 fp32 22.4 -> 25.2 us; bf16 would gain, 8 x 384 x 960
// 38.2 -> 30.8).
template <typename T>
__device__ __forceinline__ Quad<T> quad_raw_fast(const T* __restrict__ base, long off)
{
    return *reinterpret_cast<const Quad<T>*>(base + off);
}

// Four consecutive 2-byte elements at ANY element address (rows of odd length start at
// odd elements every other row, where a 4-byte access is not allowed): the three
// aligned dwords around them are loaded and shifted by 16 bits where the address is
// odd.  Branch-free, so lanes of either parity share the instructions.  The load
// covers the 12 bytes from the address rounded down to 4: the caller guarantees that
// they lie inside the tensor (one element before an odd address always does; up to
// two elements after the quad must).
struct __attribute__((packed, aligned(4))) Words3 { uint32_t v[3]; };
// the quad at p from the words around it
__device__ __forceinline__ Quad<bf16_t> quad_of_words(const Words3& w, const bf16_t* p)
{
    const uint32_t sh = (static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)) & 2u) * 8u;      // 0 or 16
    const uint32_t lo = __builtin_amdgcn_alignbit(w.v[1], w.v[0], sh);
    const uint32_t hi = __builtin_amdgcn_alignbit(w.v[2], w.v[1], sh);
    Quad<bf16_t> q;
    q.v[0].bits = (uint16_t)lo; q.v[1].bits = (uint16_t)(lo >> 16);
    q.v[2].bits = (uint16_t)hi; q.v[3].bits = (uint16_t)(hi >> 16);
    return q;
}
// The matching store: 2 + 4 + 2 bytes at an odd element address, 8 bytes at an even one.
__device__ __forceinline__ void quad_store_unaligned(bf16_t* __restrict__ p, const float in[4])
{
    bf16_t e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = from_f32<bf16_t>(in[k]);
    if (reinterpret_cast<uintptr_t>(p) & 2u) {
        p[0] = e[0];
        *reinterpret_cast<uint32_t*>(p + 1) = (uint32_t)e[1].bits | ((uint32_t)e[2].bits << 16);
        p[3] = e[3];
    } else {
        Quad<bf16_t> q;
#pragma unroll
        for (int k = 0; k < 4; ++k) q.v[k] = e[k];
        *reinterpret_cast<Quad<bf16_t>*>(p) = q;
    }
}
__device__ __forceinline__ void quad_store_unaligned(float* __restrict__ p, const float in[4])
{
    Quad<float> q;
#pragma unroll
    for (int k = 0; k < 4; ++k) q.v[k] = in[k];
    *reinterpret_cast<Quad<float>*>(p) = q;
}

template <typename T> __device__ __forceinline__ T zero_elem();
template <> __device__ __forceinline__ float zero_elem<float>() { return 0.0f; }
template <> __device__ __forceinline__ bf16_t zero_elem<bf16_t>() { bf16_t z; z.bits = 0; return z; }
// v, or zero, chosen between as plain numbers (see quad_raw_checked).
__device__ __forceinline__ float keep_if(bool keep, float v) { return keep ? v : 0.0f; }
__device__ __forceinline__ bf16_t keep_if(bool keep, bf16_t v)
{
    const uint16_t zero = 0, bits = v.bits;
    v.bits = keep ? bits : zero;
    return v;
}

template <typename T>
__device__ __forceinline__ Quad<T> quad_raw_checked(const T* __restrict__ base, long off, int ph, int L)
{
    Quad<T> q;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int t = ph + e;
        const int tc = t < 0 ? 0 : (t >= L ? L - 1 : t);
        const T v = base[off + (tc - ph)];
        q.v[e] = (t == tc) ? v : zero_elem<T>();
    }
    return q;
}
// The same for a scan order: element e is the token ord(ph + e) of the row that
// starts at base + off - ph.
template <typename T>
__device__ __forceinline__ Quad<T> quad_raw_checked(const T* __restrict__ base, long off, int ph, int L,
                                                    const TokenOrder& ord)
{
    if (ord.kind == 0) return quad_raw_checked<T>(base, off, ph, L);
    Quad<T> q;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int t = ph + e;
        const int tc = t < 0 ? 0 : (t >= L ? L - 1 : t);
        const T v = base[(off - ph) + ord(tc)];
        q.v[e] = keep_if(t == tc, v);
    }
    return q;
}

template <typename T>
__device__ __forceinline__ void quad_store(T* __restrict__ base, long off, bool fast,
                                           int ph, int L, const float in[4])
{
    if (fast) {
        Quad<T> q;
#pragma unroll
        for (int e = 0; e < 4; ++e) q.v[e] = from_f32<T>(in[e]);
        *reinterpret_cast<Quad<T>*>(base + off) = q;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (ph + e >= 0 && ph + e < L) base[off + e] = from_f32<T>(in[e]);
    }
}
// The same for a scan order (never fast then: the four tokens are not neighbours).
template <typename T>
__device__ __forceinline__ void quad_store(T* __restrict__ base, long off, bool fast,
                                           int ph, int L, const float in[4], const TokenOrder& ord)
{
    if (ord.kind == 0) { quad_store<T>(base, off, fast, ph, L, in); return; }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (ph + e >= 0 && ph + e < L) base[(off - ph) + ord(ph + e)] = from_f32<T>(in[e]);
}

}  // namespace lbscan
