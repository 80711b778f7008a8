// Offline packing, unpacking and dequantization kernels (gfx950).
//
// Quantizer: the paper fixes bits and group size only (Sec. 3.3: gate/up
// INT2, every other linear INT4, group-wise; Sec. 4.1: Stage 1 post-training
// quantization).  This library reads it as round-to-nearest asymmetric
// min-max with an integer zero point and a binary16 scale; the arithmetic is
// IEEE fp64 with exactly one rounding of the scale to binary16, so every
// code, scale and zero is reproducible bit for bit.
#include <type_traits>

#include "qmlp_device.h"
#include "qmlp_internal.h"

#pragma clang fp contract(off)

namespace qmlp {

// fp64 -> binary16 bits, a single round-to-nearest-even (never through fp32).
// Built from the bit fields of the double.
__device__ uint32_t f64_to_f16_bits(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t sign = (uint32_t)(b >> 48) & 0x8000u;
    const int e = (int)((b >> 52) & 0x7FF);
    const uint64_t frac = b & ((1ull << 52) - 1);
    if (e == 0x7FF)
        return frac ? 0x7E00u : (sign | 0x7C00u);
    if (e == 0)
        return sign;                       // fp64 subnormal: far below 2^-25
    const int E = e - 1023;                // value = 1.frac * 2^E
    if (E > 15)
        return sign | 0x7C00u;
    uint64_t keep, rest, halfway;
    int shift;
    uint64_t mant = (1ull << 52) | frac;   // 53-bit significand
    if (E >= -14) {
        shift = 42;                        // keep 11 bits (implicit one + 10)
    } else {
        shift = 42 + (-14 - E);            // subnormal: quantum 2^-24
        if (shift > 63)
            return sign;                   // below half the smallest subnormal
    }
    keep = mant >> shift;
    rest = mant & ((1ull << shift) - 1);
    halfway = 1ull << (shift - 1);
    if (rest > halfway || (rest == halfway && (keep & 1)))
        ++keep;
    if (E >= -14) {
        int he = E + 15;
        if (keep == 2048) {                // rounded up to the next binade
            keep = 1024;
            ++he;
        }
        if (he >= 31)
            return sign | 0x7C00u;
        return sign | ((uint32_t)he << 10) | (uint32_t)(keep - 1024);
    }
    return sign | (uint32_t)keep;          // keep == 1024 is 2^-14, still correct
}

__device__ double f16_bits_to_f64(uint32_t h) { return (double)h2f(h); }

// rint(w / sd) for a positive binary16 scale sd, exactly as IEEE fp64 division
// followed by rint gives it, in fp32.  w has 24 significant bits and sd 11,
// so w / sd is either a half integer exactly or at least 2^-23 of itself
// away from one, and fp64 rounding never moves it onto one: the answer is the
// integer nearest to the true quotient, ties to even.  c = rint(w * r) with
// r = fl(1 / sd) is that integer or a neighbour (the quotient's magnitude is
// at most 1.5 * 15 + 1, so the product is off by less than 1e-5), and the
// remainder w - c sd is exact in fp32: it is a multiple of the smaller of the
// two operands' last places and no larger than sd.
__device__ __forceinline__ float div_rint(float w, float sd, float r) {
    float c = __builtin_rintf(w * r);
    const float rem = __builtin_fmaf(-c, sd, w);
    const float twice = 2.0f * __builtin_fabsf(rem);
    const float next = c + __builtin_copysignf(1.0f, rem);
    const bool odd = ((int)c & 1) != 0;
    return twice > sd || (twice == sd && odd) ? next : c;
}

// Min, max and OR of `bad` over the LPG consecutive lanes of a group (8, 16
// or 32), in every lane.
template <int LPG>
__device__ __forceinline__ void group_range(float& lo, float& hi, uint32_t& bad) {
    auto step = [&](float l2, float h2, uint32_t b2) {
        lo = __builtin_fminf(lo, l2);
        hi = __builtin_fmaxf(hi, h2);
        bad |= b2;
    };
    auto d = [](uint32_t v, auto ctrl) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, false);
    };
    auto dstep = [&](auto ctrl) {
        step(__uint_as_float(d(__float_as_uint(lo), ctrl)), __uint_as_float(d(__float_as_uint(hi), ctrl)),
             d(bad, ctrl));
    };
    dstep(std::integral_constant<int, DPP_QUAD_XOR1>{});
    dstep(std::integral_constant<int, DPP_QUAD_XOR2>{});
    dstep(std::integral_constant<int, DPP_HALF_MIRROR>{});
    if constexpr (LPG >= 16)
        dstep(std::integral_constant<int, DPP_MIRROR>{});
    if constexpr (LPG >= 32)
        step(__shfl_xor(lo, 16, 64), __shfl_xor(hi, 16, 64), __shfl_xor(bad, 16, 64));
}

// Lane I of this lane's quad, to all four of them.
template <int I>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, I * 0x55, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ uint32_t or_dpp(uint32_t v) {
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// W is [n][k] fp32; codes row-major words; meta one uint32 per group: scale
// bits low, zero bits high.  At 2 and 4 bits codes, groups and weights are
// flat arrays (rows are whole words and groups).  3 bits (Appendix B): a row
// is two planes, the low two bits of every code in the 2-bit layout (k/16
// words) followed by the high bit of every code (k/32 words, code i at bit
// i mod 32 of word i/32 of the plane).
//
// What bounds it is reading W (4 bytes per weight against 0.3 to 0.7 written),
// so a wave owns 1024 consecutive weights as four 16-byte loads per lane, each
// load 1 KB contiguous, and a group is G / 4 consecutive lanes of one load.
// The range is reduced between lanes; the fp64 arithmetic of scale and zero
// (two divisions) is done once per lane for the load of its place in the
// quad and handed to the other three by quad broadcasts, so it costs one
// pass per 16 weights; the quotient of each weight is div_rint above.  Codes
// of neighbouring lanes are OR-ed into words by quad moves.
// One thread per group (a strided fp64 loop) took 3357 us for the three
// matrices of a 4096 x 12288 block (196 GB/s); this takes
// 163 us (4.0 TB/s, of 4.9 that a large copy reaches).
template <int BITS, int G>
__global__ void __launch_bounds__(256)
pack_kernel(const float* __restrict__ W, long total, int k, uint32_t* __restrict__ codes,
            uint32_t* __restrict__ meta, int32_t* status) {
    constexpr int QMAX = (1 << BITS) - 1;
    constexpr int LPG = G / 4;                            // lanes per group of one load
    const int lane = threadIdx.x & 63;
    const long base = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 1024;
    if (base >= total)
        return;
    u32x4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const long e = base + 256 * i + 4 * lane;         // a group is inside total or past it as a whole
        v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(W + (e < total ? e : 0)));
    }
    float lo = 0.0f, hi = 0.0f;                           // of the load of this lane's place in its quad
    uint32_t bad = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float l = 0.0f, h = 0.0f;
        uint32_t b = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t u = v[i][j];
            const bool fin = (u & 0x7F800000u) != 0x7F800000u;
            const float f = fin ? __uint_as_float(u) : 0.0f;
            l = __builtin_fminf(l, f);
            h = __builtin_fmaxf(h, f);
            b |= fin ? 0u : 1u;
        }
        group_range<LPG>(l, h, b);
        if ((lane & 3) == i) {
            lo = l;
            hi = h;
            bad = b;
        }
    }
    const double s = ((double)hi - (double)lo) / (double)QMAX;
    uint32_t s16 = f64_to_f16_bits(s);
    if (s16 == 0)
        s16 = 0x3C00u;                                    // degenerate range: scale 1.0
    const bool invalid = bad != 0 || s16 == 0x7C00u;
    const double sd64 = f16_bits_to_f64(s16);
    double zf = __builtin_rint(-(double)lo / sd64);
    zf = zf < 0.0 ? 0.0 : (zf > (double)QMAX ? (double)QMAX : zf);
    const float z1 = invalid ? 0.0f : (float)(int)zf;         // through int: never -0
    const uint32_t m1 = invalid ? 0x00007E00u : s16 | (f2h(z1) << 16);   // invalid: scale NaN, zero 0
    const float r1 = 1.0f / h2f(s16);

    // codes of the four weights of each load
    uint32_t q[4], qh[4];
    auto load_codes = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const uint32_t m = quad_bcast<i>(m1);
        const float r = __uint_as_float(quad_bcast<i>(__float_as_uint(r1)));
        const float sd = h2f(m & 0xFFFFu), z = h2f(m >> 16);
        const bool ok = (m & 0xFFFFu) != 0x7E00u;
        uint32_t word = 0, high = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float t = div_rint(__uint_as_float(v[i][j]), sd, r) + z;
            const uint32_t c = ok ? (uint32_t)__builtin_fminf(__builtin_fmaxf(t, 0.0f), (float)QMAX) : 0u;
            if (BITS == 3) {
                word |= (c & 3u) << (2 * j);
                high |= (c >> 2) << j;
            } else {
                word |= c << (BITS * j);
            }
        }
        q[i] = word;
        qh[i] = high;
        const long e = base + 256 * i + 4 * lane;
        if (lane % LPG == 0 && e < total) {
            meta[e / G] = m;
            if (!ok && status)
                atomicOr(status, 1);
        }
    };
    load_codes(std::integral_constant<int, 0>{});
    load_codes(std::integral_constant<int, 1>{});
    load_codes(std::integral_constant<int, 2>{});
    load_codes(std::integral_constant<int, 3>{});

    const int p = lane & 3, quad = lane >> 2;
    if constexpr (BITS == 4) {
        // a word is the halves of two lanes; lane p of a quad keeps load p's two words
        uint32_t a = 0, b = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = or_dpp<DPP_QUAD_XOR1>(q[i] << (16 * (lane & 1)));
            const uint32_t w0 = quad_bcast<0>(w), w1 = quad_bcast<2>(w);
            if (p == i) {
                a = w0;
                b = w1;
            }
        }
        const long e = base + 256 * p + 16 * quad;        // first code of the two words
        if (e < total)
            *reinterpret_cast<uint2*>(codes + e / 8) = make_uint2(a, b);
    } else {
        // a word is the bytes of a quad; lane p of a quad keeps load p's word
        uint32_t a = 0, h = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = or_dpp<DPP_QUAD_XOR2>(or_dpp<DPP_QUAD_XOR1>(q[i] << (8 * p)));
            if (p == i)
                a = w;
            if constexpr (BITS == 3) {
                // the high plane's word is the nibbles of eight lanes
                const uint32_t x = or_dpp<DPP_HALF_MIRROR>(
                    or_dpp<DPP_QUAD_XOR2>(or_dpp<DPP_QUAD_XOR1>(qh[i] << (4 * (lane & 7)))));
                if (p == i)
                    h = x;
            }
        }
        const long e = base + 256 * p + 16 * quad;        // first code of the word
        if (e < total) {
            if constexpr (BITS == 2) {
                codes[e / 16] = a;
            } else {
                const long row = e / k, col = e - row * k;
                uint32_t* out = codes + row * ((long)k * 3 / 32);
                out[col / 16] = a;
                if ((quad & 1) == 0)
                    out[k / 16 + col / 32] = h;
            }
        }
    }
}

// One thread per 32-bit code word: canonical codes uint8 [n][k]; the thread
// holding the first word of a group also writes that group's scale and zero.
// Code i of a word: BITS-bit field i; at 3 bits the 2-bit field of the low
// plane and the bit of the high plane (code_word: the low-plane word, hi:
// the high-plane bits of the same 16 codes, in bits 0-15).
template <int BITS>
__device__ __forceinline__ uint32_t code_at(uint32_t code_word, uint32_t hi, int i) {
    if (BITS == 3)
        return ((code_word >> (2 * i)) & 3u) | (((hi >> i) & 1u) << 2);
    return (code_word >> (BITS * i)) & ((1u << BITS) - 1);
}

// The word of the (low) plane at word index gid of the row-major view, the
// row and first code column it covers, and the matching high-plane bits.
template <int BITS>
__device__ __forceinline__ void word_at(const uint32_t* codes, int k, long gid, uint32_t& wv,
                                        uint32_t& hi, long& row, long& col) {
    constexpr int PER = BITS == 3 ? 16 : 32 / BITS;
    row = gid / (k / PER);
    col = (gid - row * (k / PER)) * PER;
    const long row_words = BITS == 3 ? (long)k * 3 / 32 : (long)(k / PER);
    wv = codes[row * row_words + col / PER];
    hi = BITS == 3 ? codes[row * row_words + k / 16 + col / 32] >> (col & 31) : 0u;
}

template <int BITS>
__global__ void __launch_bounds__(256)
unpack_kernel(const uint32_t* __restrict__ codes, const uint32_t* __restrict__ meta,
              int n, int k, int g, uint8_t* __restrict__ out_codes,
              uint16_t* __restrict__ scales, uint16_t* __restrict__ zeros) {
    constexpr int PER = BITS == 3 ? 16 : 32 / BITS;
    const long words = (long)n * (k / PER);
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= words)
        return;
    uint32_t w, hi;
    long row, col;                                    // col: first code index in the row
    word_at<BITS>(codes, k, gid, w, hi, row, col);
    uint8_t* dst = out_codes + row * (long)k + col;
    for (int i = 0; i < PER; ++i)
        dst[i] = (uint8_t)code_at<BITS>(w, hi, i);
    if (col % g == 0) {
        const long gi = row * (k / g) + col / g;
        const uint32_t m = meta[gi];
        scales[gi] = (uint16_t)(m & 0xFFFFu);
        zeros[gi] = (uint16_t)(m >> 16);
    }
}

// One thread per code word: w_hat = scale * (q - zero) is exact in fp32
// (an 11-bit scale times an integer below 16), then one nearest-even
// rounding to binary16.  A NaN scale (invalid group) yields 0x7E00.
template <int BITS>
__global__ void __launch_bounds__(256)
dequant_kernel(const uint32_t* __restrict__ codes, const uint32_t* __restrict__ meta,
               int n, int k, int g, uint16_t* __restrict__ out) {
    constexpr int PER = BITS == 3 ? 16 : 32 / BITS;
    const long words = (long)n * (k / PER);
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= words)
        return;
    uint32_t w, hi;
    long row, col;
    word_at<BITS>(codes, k, gid, w, hi, row, col);
    const uint32_t m = meta[row * (k / g) + col / g];
    const float s = h2f(m & 0xFFFFu);
    const float z = h2f(m >> 16);
    const bool nan_scale = (m & 0x7C00u) == 0x7C00u && (m & 0x03FFu) != 0;
    uint16_t* dst = out + row * (long)k + col;
    for (int i = 0; i < PER; ++i) {
        const float q = (float)code_at<BITS>(w, hi, i);
        const float v = s * (q - z) + 0.0f;
        dst[i] = nan_scale ? (uint16_t)0x7E00u : (uint16_t)f2h(v);
    }
}

static inline unsigned blocks_for(long threads) { return (unsigned)((threads + 255) / 256); }

template <int BITS>
static void pack_bits(const float* W, long total, int k, int g, uint32_t* codes, uint32_t* meta,
                      int32_t* status, hipStream_t st) {
    const unsigned grid = (unsigned)((total + 4095) / 4096);       // four waves of 1024 weights
    if (g == 32)
        pack_kernel<BITS, 32><<<grid, 256, 0, st>>>(W, total, k, codes, meta, status);
    else if (g == 64)
        pack_kernel<BITS, 64><<<grid, 256, 0, st>>>(W, total, k, codes, meta, status);
    else
        pack_kernel<BITS, 128><<<grid, 256, 0, st>>>(W, total, k, codes, meta, status);
}

hipError_t launch_pack(int bits, const float* W, int n, int k, int g, uint32_t* codes,
                       uint32_t* meta, int32_t* status, hipStream_t st) {
    const long total = (long)n * k;
    if (bits == 2)
        pack_bits<2>(W, total, k, g, codes, meta, status, st);
    else if (bits == 3)
        pack_bits<3>(W, total, k, g, codes, meta, status, st);
    else
        pack_bits<4>(W, total, k, g, codes, meta, status, st);
    return hipGetLastError();
}

hipError_t launch_unpack(int bits, const uint32_t* codes, const uint32_t* meta, int n, int k,
                         int g, uint8_t* out_codes, uint16_t* scales, uint16_t* zeros,
                         hipStream_t st) {
    const long words = (long)n * (k / (bits == 4 ? 8 : 16));
    if (bits == 2)
        unpack_kernel<2><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out_codes,
                                                             scales, zeros);
    else if (bits == 3)
        unpack_kernel<3><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out_codes,
                                                             scales, zeros);
    else
        unpack_kernel<4><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out_codes,
                                                             scales, zeros);
    return hipGetLastError();
}

hipError_t launch_dequant(int bits, const uint32_t* codes, const uint32_t* meta, int n, int k,
                          int g, uint16_t* out, hipStream_t st) {
    const long words = (long)n * (k / (bits == 4 ? 8 : 16));
    if (bits == 2)
        dequant_kernel<2><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out);
    else if (bits == 3)
        dequant_kernel<3><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out);
    else
        dequant_kernel<4><<<blocks_for(words), 256, 0, st>>>(codes, meta, n, k, g, out);
    return hipGetLastError();
}

}  // namespace qmlp
