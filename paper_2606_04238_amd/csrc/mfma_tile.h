// Device helpers shared by the matrix-core decode kernels (decode_mfma.hip,
// decode_tile.hip): the 16x16x32 step, buffer loads, and the whole-line
// weight loads with the register moves into the matrix layout.
#pragma once

#include "decode_common.h"

namespace qmlp {
namespace {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef const BatchArgs __attribute__((address_space(4))) KBatchM;
__device__ __forceinline__ KBatchM* kbm() { return (KBatchM*)__builtin_amdgcn_kernarg_segment_ptr(); }

__device__ __forceinline__ f32x4_t mfma16(const uint4& a, const uint4& b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a),
                                                  __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

// Lanes 32-63 of a trade places with lanes 0-31 of b.
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
// Lanes 16-31 and 48-63 of a trade places with lanes 0-15 and 32-47 of b.
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// LDS barrier that leaves vector-memory loads in flight: this wave's LDS
// accesses complete, then the workgroup meets.
__device__ __forceinline__ void lds_barrier() {
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Weight loads go through buffer resources: a resource of zero bytes turns
// a load into one that returns zeros without touching memory, so a prefetch
// that has nothing to fetch issues the same instructions as one that has
// (the compiler then keeps the next step's loads in flight across a step),
// and every load is bounds-checked against its array.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
constexpr int kAuxNt = 2;      // non-temporal: codes are read once
constexpr int kAuxDevice = 16; // device-coherent (sc1): written by another compute unit in this launch
template <int AUX>
__device__ __forceinline__ uint4 bload16(Rsrc r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, AUX);
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ uint2 bload8(Rsrc r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return make_uint2(v[0], v[1]);
}

// Whole-line loads.  A step reads 128 bytes (eight 16-byte units) of each of
// 16 weight rows; each load instruction covers 8 rows whole (lane L: row
// 8 h + (L & 7) for load h, unit u(L) from lane bits 5..3), so every 128-byte
// line is fetched by one instruction.  The matrix cores want lane l = 16 q + j
// to hold row j, so the units are then moved between lanes in registers: with
// the row bit h exchanged for lane bit 3 (E3, a row rotation by 8 under a
// bank mask), the 4-byte words of a unit u = (u2 u1 u0), w = (w1 w0) sit at
// register (u2 after E3) and component (w1 w0); E4 exchanges lane bit 4 with
// component bit w1 (v_permlane16_swap) and E5 lane bit 5 with w0
// (v_permlane32_swap).  Which unit bit each lane bit carries is chosen per
// layout so that a quarter's words of one group end up in the same register
// positions for every group (QW words per quarter and group):
//   2-bit g = 128, 4-bit g = 64 (E3, E4): lane bits 5, 4, 3 = u0, u1, u2;
//     quarter q holds words 2q, 2q + 1 of a group;
//   2-bit g = 64 (E3, E4, E5): same units; quarter q holds word
//     2 (q & 1) + (q >> 1) of each group;
//   4-bit g = 128 (E3): lane bits 5, 4, 3 = u1, u0, u2; quarter q holds
//     words 4q .. 4q + 3.
template <int QW>
__device__ __forceinline__ int quarter_word(int q) {
    if constexpr (QW == 1) return 2 * (q & 1) + (q >> 1);
    else if constexpr (QW == 2) return 2 * q;
    else return 4 * q;
}
// 16-byte unit of the step's 128 bytes that lane L loads.
template <bool DN128>
__device__ __forceinline__ int lane_unit(int L) {
    const int b5 = (L >> 5) & 1, b4 = (L >> 4) & 1, b3 = (L >> 3) & 1;
    return DN128 ? 4 * b3 + 2 * b5 + b4 : 4 * b3 + 2 * b4 + b5;
}
constexpr int kDppRowRor8 = 0x128;
// E3 on one component: a (h = 0) and b (h = 1) become the S3 = 0 and S3 = 1
// halves, rows 8..15 taken from lane l ^ 8.
__device__ __forceinline__ void e3(uint32_t& a, uint32_t& b) {
    const int na = __builtin_amdgcn_update_dpp((int)a, (int)b, kDppRowRor8, 0xF, 0xC, false);
    const int nb = __builtin_amdgcn_update_dpp((int)b, (int)a, kDppRowRor8, 0xF, 0x3, false);
    a = (uint32_t)na;
    b = (uint32_t)nb;
}
// The exchanges of a step's two loads: E3 always, E4 and E5 as asked.
template <bool E4, bool E5>
__device__ __forceinline__ void arrange(uint4 (&v)[2]) {
    e3(v[0].x, v[1].x);
    e3(v[0].y, v[1].y);
    e3(v[0].z, v[1].z);
    e3(v[0].w, v[1].w);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (E4) {
            swap16(v[i].x, v[i].z);
            swap16(v[i].y, v[i].w);
        }
        if constexpr (E5) {
            swap32(v[i].x, v[i].y);
            swap32(v[i].z, v[i].w);
        }
    }
}

__device__ __forceinline__ uint32_t word_of(const uint4& v, int i) {
    return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

// A buffer offset past the end of every resource: the load returns zeros.
constexpr uint32_t kPastEnd = 0x80000000u;

}  // namespace
}  // namespace qmlp
