// What the wave-tile kernels share: a wave owns R rows (channels of one batch entry: 8 in the
// forward kernel, 16 in the backward one) and keeps a tile of them in LDS that no other wave
// reads, so that nothing but the shared Bm / Cm tile needs a block barrier.
//
// Two layouts of the 64 lanes meet in a tile:
//   staging:  lane = 64 / R * row + quad   four tokens of one row, as memory holds them
//   scan:     lane = R * group + row       a share (1 in 64 / R) of the row's states, all its tokens
//             (forward kernel, where Eq. 8 is summed: the eight lanes of a row within sixteen)
#pragma once
#include <type_traits>

#include "lbscan_device.h"

namespace lbscan {

constexpr int kBlockWaves = 4;                    // waves of a block (they share Bm / Cm)
constexpr int kWaveRows = 16;                     // backward kernel: rows of a wave
constexpr int kBlockRows = kWaveRows * kBlockWaves;

// LDS traffic between the lanes of one wave: the hardware keeps a wave's accesses in
// order, the compiler has to be told.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void lds_get4(const float* a, int o, float (&v)[4])
{
    const float4 q = *reinterpret_cast<const float4*>(a + o);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
__device__ __forceinline__ void lds_get8(const float* a, int o, float (&v)[8])
{
    float lo[4], hi[4];
    lds_get4(a, o, lo);
    lds_get4(a, o + 4, hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
}
__device__ __forceinline__ void lds_put4(float* a, int o, const float (&v)[4])
{
    *reinterpret_cast<float4*>(a + o) = make_float4(v[0], v[1], v[2], v[3]);
}

// How the quads of a tile come from memory (uniform over the block).
//   quads:     whole quads inside the rows
//   unaligned: the same for 2-byte rows that start at odd elements: the three aligned
//              words around a quad
//   clamped:   the ragged last tile: whole quads from the nearest position inside the row
//   tail:      a short last tile of the forward kernel: one token a lane
//   elements:  element by element (scan orders that gather, short and odd ragged rows)
enum class TileLoads { quads, unaligned, clamped, tail, elements };

// A quad as loaded.  Nothing touches it before it is needed: a conversion, or the shift of
// unaligned words, at the load would make the wave wait for it there.
// (Vectors: of single elements the compiler makes copies where ways of loading meet, and waits
// for the load to make them.)
typedef float Float4 __attribute__((ext_vector_type(4)));
typedef uint32_t Word3 __attribute__((ext_vector_type(3)));
typedef Float4 Float4At4 __attribute__((aligned(4)));        // at any 4-byte address
template <typename T> struct HeldQuad;
template <> struct HeldQuad<float> { Float4 q; };
template <> struct HeldQuad<bf16_t> { Word3 w; };

struct __attribute__((packed, aligned(4))) Words2 { uint32_t v[2]; };

// Uniform base, 32-bit byte offset per lane (the addressing form that takes no vector
// instruction).
template <typename T>
__device__ __forceinline__ const T* at_bytes(const T* base, unsigned bytes)
{
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}
template <typename T>
__device__ __forceinline__ T* at_bytes(T* base, unsigned bytes)
{
    return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + bytes);
}

__device__ __forceinline__ void hold_quad(HeldQuad<float>& h, const float* p) { h.q = *reinterpret_cast<const Float4At4*>(p); }
__device__ __forceinline__ void hold_quad(HeldQuad<bf16_t>& h, const bf16_t* p)
{
    const Words2 w = *reinterpret_cast<const Words2*>(p);
    Word3 v;                                          // (the third word is not looked at: shift 0)
    v[0] = w.v[0]; v[1] = w.v[1];
    h.w = v;
}
__device__ __forceinline__ void hold_unaligned(HeldQuad<float>& h, const float* p) { hold_quad(h, p); }
__device__ __forceinline__ void hold_unaligned(HeldQuad<bf16_t>& h, const bf16_t* p)
{
    const Words3 w = *reinterpret_cast<const Words3*>(p - ((reinterpret_cast<uintptr_t>(p) >> 1) & 1));
    h.w = Word3{w.v[0], w.v[1], w.v[2]};
}
__device__ __forceinline__ void hold_elements(HeldQuad<float>& h, const Quad<float>& q) { h.q = Float4{q.v[0], q.v[1], q.v[2], q.v[3]}; }
__device__ __forceinline__ void hold_elements(HeldQuad<bf16_t>& h, const Quad<bf16_t>& q)
{
    h.w = Word3{(uint32_t)q.v[0].bits | ((uint32_t)q.v[1].bits << 16), (uint32_t)q.v[2].bits | ((uint32_t)q.v[3].bits << 16), 0u};
}
// The quad is waited for here, on every path that may have loaded it.
__device__ __forceinline__ void arrived(const HeldQuad<float>& h) { asm volatile("" : : "v"(h.q)); }
__device__ __forceinline__ void arrived(const HeldQuad<bf16_t>& h) { asm volatile("" : : "v"(h.w)); }

// One element, first in the quad (tail).
__device__ __forceinline__ void hold_element(HeldQuad<float>& h, const float* p) { Float4 v; v[0] = *p; h.q = v; }
__device__ __forceinline__ void hold_element(HeldQuad<bf16_t>& h, const bf16_t* p) { Word3 v; v[0] = p->bits; h.w = v; }
__device__ __forceinline__ float open_element(const HeldQuad<float>& h) { return h.q[0]; }
__device__ __forceinline__ float open_element(const HeldQuad<bf16_t>& h) { return __uint_as_float(h.w[0] << 16); }

// The four elements in 32 bits, in logical order (REV: the stored order mirrored).  shift:
// 16 where the quad was held unaligned at an odd element, else 0 (2-byte types).
template <bool REV>
__device__ __forceinline__ void open_quad(const HeldQuad<float>& h, unsigned, float (&v)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) v[REV ? 3 - e : e] = h.q[e];
}
template <bool REV>
__device__ __forceinline__ void open_quad(const HeldQuad<bf16_t>& h, unsigned shift, float (&v)[4])
{
    const uint32_t lo = __builtin_amdgcn_alignbit(h.w[1], h.w[0], shift);
    const uint32_t hi = __builtin_amdgcn_alignbit(h.w[2], h.w[1], shift);
    v[REV ? 3 : 0] = __uint_as_float(lo << 16);
    v[REV ? 2 : 1] = __uint_as_float(lo & 0xffff0000u);
    v[REV ? 1 : 2] = __uint_as_float(hi << 16);
    v[REV ? 0 : 3] = __uint_as_float(hi & 0xffff0000u);
}
// A quad held from a clamped position: in logical order, wanted element e is loaded element
// e + s where 0 <= e + s < 4 (s: tokens that the position was moved by), nothing elsewhere.
__device__ __forceinline__ void move_clamped(float (&v)[4], int s)
{
    float r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float w = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) w = (e + s == j) ? v[j] : w;
        r[e] = w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = r[e];
}

// A value whose origin the compiler does not see: what is computed from it is neither moved
// out of a loop nor kept for later.
__device__ __forceinline__ int per_lane(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// A sum that is to be finished where it stands: left alone, the compiler moves the last
// additions to where the sum is used, much later, and holds their terms until then.
__device__ __forceinline__ float keep_here(float v)
{
    asm volatile("" : "+v"(v));
    return v;
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xF, 0xF, false));
}

// Sums over the 16 lanes of a row of lanes of 8 values per lane: every lane r of the 16
// ends with the sum of value r / 2.  Halving steps: the lanes with bit 3 of r set take
// over values 4..7 of both partners, then those with bit 2 the upper two of what is left;
// a DPP add reads the partner's value itself and writes only the banks it is meant for, so
// a step costs two instructions per pair of values and no select.  (The compiler does not look into the
// block: the s_nop at its ends and before the quad steps are the two wait states between
// a vector write and a DPP read of the same register.)
__device__ __forceinline__ float row16_sum8(float (&v)[8], bool bit1)
{
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3])
        : "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
    const float y = bit1 ? v[1] : v[0];
    return y + dpp_move<0xB1>(y);                 // quad_perm [1,0,3,2]
}

// Sums over the four state groups (lanes 16 apart) of four values per lane: lane group s
// ends with the sum of value s.
__device__ __forceinline__ float groups_sum4(const float (&v)[4])
{
    float w[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {                 // lanes < 32 keep values 0, 1, the others 2, 3
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 2]), false, false);
        w[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(w[0]), __float_as_uint(w[1]), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums over eight state groups (bits 1 to 3 of the lane) of four values per lane: the lanes with
// s in bits 2 and 3 end with the sum of value s.  Halving steps as in row16_sum8, within a row
// of lanes throughout: a DPP add takes half the time of a swap between rows (4 and 8 clocks a
// wave; a plain add 2).
__device__ __forceinline__ float groups8_sum4(float (&v)[4])
{
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
        : "+&v"(v[0]), "+&v"(v[1])
        : "v"(v[2]), "v"(v[3]));
    return v[0];
}

}  // namespace lbscan
