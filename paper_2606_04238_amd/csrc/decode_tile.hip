// Decode at several tokens (M <= 16, binary16) on the matrix cores at every
// group of 2- and 4-bit codes, gfx950: the gate/up half with rows of at most
// twelve steps (2 bits d <= 6144, 4 bits d <= 3072; Sec. 3.1 Eq. (1), Sec. 3.3,
// Sec. 4.2, Sec. 5) and any quantized linear (Sec. 3.3).
//
// What bounds it.  On the vector ALU a weight costs M/2 dot2 operations on
// top of its unpacking, so from a few tokens on the stand-alone kernels are
// bound by arithmetic (a Qwen3-8B-shaped block at M = 8: 107 us for 57 MB).
// Here a weight is unpacked once and multiplied into all tokens by
// v_mfma_f32_16x16x32_f16, so the weight stream is the bound again.
//
// Split.  A workgroup's waves split K: wave kw owns SPW steps of 128 bytes
// per weight row (1024 / B codes each) and keeps the activations of those
// steps IN REGISTERS as matrix operands (the tokens as the 16 rows) for all
// the 16-row tiles its workgroup walks.  The inner loop then reads nothing
// but weights from memory and the per-group sums below from LDS: a layout
// that keeps the activations in LDS reads 1 KB of them per 128 bytes of 2-bit
// weights, which at these rates is LDS bandwidth.  The waves' partial sums of
// a tile meet in LDS (double-buffered, one barrier per tile that leaves the
// weight prefetch in flight) and one wave, another one each tile, adds them
// and writes the outputs.  Where K is short, TW groups of waves take tiles
// side by side; where it is too long for the registers of one workgroup, SK
// workgroups take a slice each of a range of tiles and leave fp32 partials,
// and the last of them to finish (a counter per range) adds the slices in
// order.  No workgroup waits for another.
//
// The arithmetic: codes enter as 1024 + q 2^j (one and-or per pair; j >= 4,
// so that the offset's share of the fp32 sums and their rounding stays small:
// at j from 0 the error against 64 bits was 2 % larger) and the activation as
// x' = x 2^(4 - j), so a code's product is 1024 x' + 16 q x and a tile's
// finished sum is multiplied by 2^-4 once.  (With x 2^-j the factor is not
// needed, but x' is binary16 and small activations lose more bits below its
// normal range: a 4-bit linear on inputs of rms 6e-4 was 1.3e-3 off 64 bits
// instead of 2.1e-4, and a 2-bit one 3.9e-3 instead of 3.2e-4, in a CPU model
// of the operands.)  The products'
// offset and the zero point come off as an fp32 contraction over the groups
// of s and s z with C = 1024 sum x' and X = 16 sum x (formed on the matrix
// cores as products with constants, which leaves them in the operand's own
// layout), and a group adds scale * (its product) in fp32.
// LoRA-B stays fp32: t is the A operand and B (exact in fp32) the B operand
// of v_mfma_f32_16x16x4_f32, four ranks per instruction.
//
// Lane l = 16 q + j holds weight row j of the tile; see decode_mfma.hip for
// the whole-line loads and the register moves that bring quarter q its words
// of every group.  2-bit groups of 32 are two words, too few for four
// quarters: a lane trades words with the neighbouring quarter
// (v_permlane16_swap) so that quarters 2 w and 2 w + 1 hold word w of both
// groups of a 16-byte unit and take its codes 0..7 and 8..15.
#include "decode_common.h"
#include "decode_launch.h"
#include "mfma_tile.h"
#include "tile_plan.h"

namespace qmlp {

static_assert(kTileBatch == kBatchMax, "one batch size");

namespace {

// The same value, opaque to the compiler: addresses formed from it where they
// are used now and then (once per block or tile) are not kept across the main
// loop, which has no register to spare.
__device__ __forceinline__ int fresh(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Layout of one step (32 code words of each of 16 rows) of B-bit codes in
// groups of G.
template <int B, int G>
struct Lay {
    static constexpr int CPS = 1024 / B;                   // codes per row and step
    static constexpr int WPG = G * B / 32;                 // words per group
    static constexpr bool HALF = WPG == 2;                 // 2-bit, group 32
    static constexpr int QW = HALF ? 1 : WPG / 4;          // words per quarter and group
    static constexpr int GSU = 32 / WPG;                   // groups per step
    static constexpr int MPG = HALF ? 1 : B == 2 ? 2 * QW : QW;   // matrix instructions per group
    static constexpr int NA = MPG * GSU;                   // A operands per step
};

template <int B, int G>
using AOps = uint4[Lay<B, G>::NA];

// The (scale | zero) words of a step's groups of lane row j: quarter q loads
// its quarter of them, groups q GSU/4 .. (both where there are only two), and
// meta_spread hands them to the other quarters.
template <int GSU>
struct TileMeta {
    static constexpr int NW = GSU == 2 ? 2 : GSU / 4;
    uint32_t w[NW];
};
template <int GSU>
__device__ __forceinline__ int meta_first(int q) { return GSU == 2 ? 0 : q * (GSU / 4); }
template <int GSU>
__device__ __forceinline__ void meta_load(TileMeta<GSU>& m, Rsrc r, uint32_t voff) {
    if constexpr (GSU == 16) {
        const uint4 v = bload16<0>(r, voff, 0);
        m.w[0] = v.x;
        m.w[1] = v.y;
        m.w[2] = v.z;
        m.w[3] = v.w;
    } else if constexpr (GSU == 4) {
        m.w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0);
    } else {
        const uint2 v = bload8(r, voff, 0);
        m.w[0] = v.x;
        m.w[1] = v.y;
    }
}
// Word e of every quarter, in all quarters: sc[k] is the scale of group
// k GSU/4 + e (with equal operands a swap leaves one side's value on both).
__device__ __forceinline__ void meta_spread(uint32_t w, float (&sc)[4]) {
    uint32_t x = w, y = w;
    swap16(x, y);                                          // x: quarters 0 0 2 2, y: 1 1 3 3
    uint32_t x2 = x, y2 = y;
    swap32(x, x2);                                         // x: 0 everywhere, x2: 2
    swap32(y, y2);
    sc[0] = h2f(x & 0xFFFFu);
    sc[1] = h2f(y & 0xFFFFu);
    sc[2] = h2f(x2 & 0xFFFFu);
    sc[3] = h2f(y2 & 0xFFFFu);
}

// ---- activations
// Raw activations of (this lane's) step gs: token j (zeros past M) and the
// words of its quarter (zeros past K; `live` false: all zeros).  rx covers
// the block's M rows of K.
template <int B, int G>
__device__ __forceinline__ void act_load(AOps<B, G>& a, Rsrc rx, int gs, int j, int M, int K, bool live, int lane) {
    typedef Lay<B, G> Y;
    constexpr int CW = 32 / B;                             // codes per word
    const int q = lane >> 4;
    const bool tok = live && j < M;
    const int W0 = gs * 32 + (Y::HALF ? q >> 1 : quarter_word<Y::QW>(q));
    const uint32_t o = tok ? (uint32_t)(j * K + CW * W0 + (Y::HALF ? 8 * (q & 1) : 0)) * 2u : kPastEnd;
    constexpr int NWD = Y::HALF ? Y::GSU : Y::GSU * Y::QW;
#pragma unroll
    for (int i = 0; i < NWD; ++i) {
        const uint32_t oi = o + 2u * CW * (Y::HALF ? 2 * i : (i / Y::QW) * Y::WPG + i % Y::QW);
        if constexpr (B == 2 && !Y::HALF) {
            a[2 * i] = bload16<0>(rx, oi, 0);
            a[2 * i + 1] = bload16<0>(rx, oi + 16, 0);
        } else {
            a[i] = bload16<0>(rx, oi, 0);
        }
    }
}
// Words past the row's end (the next token's) become zeros.
template <int B, int G>
__device__ __forceinline__ void act_mask(AOps<B, G>& a, int gs, int K, int lane) {
    typedef Lay<B, G> Y;
    constexpr int CW = 32 / B, PER = Y::HALF || B == 4 ? 1 : 2;
    if (__all((gs + 1) * Y::CPS <= K))
        return;
    const int q = lane >> 4, W0 = gs * 32 + (Y::HALF ? q >> 1 : quarter_word<Y::QW>(q));
#pragma unroll
    for (int i = 0; i < Y::NA; ++i) {
        const int k = i / PER;
        if (CW * (W0 + (Y::HALF ? 2 * k : (k / Y::QW) * Y::WPG + k % Y::QW)) >= K)
            a[i] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// (a.lo, b.lo) and (a.hi, b.hi) of two words of halves.
__device__ __forceinline__ uint32_t pair_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pair_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ uint32_t pk_mul(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) * __builtin_bit_cast(half2_t, b));
}
__device__ __forceinline__ constexpr uint32_t pow2_pair(int e) {      // binary16 2^e in both halves
    return (uint32_t)((15 + e) << 10) * 0x00010001u;
}
// Fraction position j of pair p (0..3) of the matrix operand of half h, and
// the smallest of them: x' = x 2^(kPosMin - j).
constexpr int kPosMin = 4;
constexpr float kTileUnscale = 1.0f / 16.0f;               // 2^-kPosMin, of a finished sum
template <int B, bool HALF>
__device__ __forceinline__ constexpr int pair_pos(int h, int p) {
    if (B == 4) return p < 2 ? 4 : 6;
    if (HALF || h == 0) return (p & 1) ? 6 : 4;
    return p == 1 ? 4 : p == 2 ? 6 : 8;
}
template <int B, bool HALF>
__device__ __forceinline__ uint4 scale_pairs(uint4 v, int h) {
    return make_uint4(pk_mul(v.x, pow2_pair(kPosMin - pair_pos<B, HALF>(h, 0))),
                      pk_mul(v.y, pow2_pair(kPosMin - pair_pos<B, HALF>(h, 1))),
                      pk_mul(v.z, pow2_pair(kPosMin - pair_pos<B, HALF>(h, 2))),
                      pk_mul(v.w, pow2_pair(kPosMin - pair_pos<B, HALF>(h, 3))));
}
template <int B, bool HALF>
__device__ __forceinline__ uint4 unscale_pairs(int h) {
    return make_uint4(pow2_pair(pair_pos<B, HALF>(h, 0)), pow2_pair(pair_pos<B, HALF>(h, 1)),
                      pow2_pair(pair_pos<B, HALF>(h, 2)), pow2_pair(pair_pos<B, HALF>(h, 3)));
}
// Raw words to matrix operands x' in the pair order of the codes.
template <int B, int G>
__device__ __forceinline__ void act_convert(AOps<B, G>& a) {
    typedef Lay<B, G> Y;
    if constexpr (B == 2 && !Y::HALF) {
#pragma unroll
        for (int i = 0; i < Y::NA / 2; ++i) {
            const uint4 l = a[2 * i], h = a[2 * i + 1];
            a[2 * i] = scale_pairs<B, false>(make_uint4(pair_lo(l.x, h.x), pair_hi(l.x, h.x), pair_lo(l.y, h.y),
                                                        pair_hi(l.y, h.y)), 0);
            a[2 * i + 1] = scale_pairs<B, false>(make_uint4(pair_lo(l.z, h.z), pair_hi(l.z, h.z), pair_lo(l.w, h.w),
                                                            pair_hi(l.w, h.w)), 1);
        }
    } else {
#pragma unroll
        for (int i = 0; i < Y::NA; ++i) {                  // eight codes, pairs p and 4 + p
            const uint4 r = a[i];
            a[i] = scale_pairs<B, Y::HALF>(make_uint4(pair_lo(r.x, r.z), pair_hi(r.x, r.z), pair_lo(r.y, r.w),
                                                    pair_hi(r.y, r.w)), 0);
        }
    }
}
// The A operands of a step's offset and zero-point terms.  With C = sum x'
// and X = sum 2^j x' (16 sum x) of a token and group, the group's codes add
// s (p - 1024 C - z X), p their plain product with x'.  The second and third
// terms of all groups are one fp32 contraction over groups, rows (s, s z)
// against tokens (-1024 C, -X): v_mfma_f32_16x16x4_f32, where instruction m
// takes the m-th group of every quarter of the lanes, whose words that quarter
// loaded (two groups per step: quarters 0, 1 the C and 2, 3 the X of groups
// 0, 1).  C and X come from the matrix cores with the activations as the B
// operand, so every lane gets its own token's.
template <int B, int G>
struct Corr {
    static constexpr int NC = Lay<B, G>::GSU == 2 ? 1 : Lay<B, G>::GSU / 4;
    float c[NC], x[NC];
};
template <int B, int G>
__device__ __forceinline__ void group_sums(const AOps<B, G>& a, Corr<B, G>& k, int lane) {
    typedef Lay<B, G> Y;
    const uint4 one = make_uint4(0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u);
    const int q = lane >> 4;
#pragma unroll
    for (int i = 0; i < Y::GSU; ++i) {
        f32x4_t c = {0.f, 0.f, 0.f, 0.f}, x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < Y::MPG; ++m) {
            c = mfma16(one, a[i * Y::MPG + m], c);
            x = mfma16(unscale_pairs<B, Y::HALF>(B == 2 && !Y::HALF ? m & 1 : 0), a[i * Y::MPG + m], x);
        }
        if constexpr (Y::GSU == 2) {
            if (i == 0 || (q & 1)) k.c[0] = q < 2 ? -1024.0f * c[0] : -x[0];
        } else {
            constexpr int NC = Corr<B, G>::NC;
            if (i < NC || q == i / NC) {
                k.c[i % NC] = -1024.0f * c[0];
                k.x[i % NC] = -x[0];
            }
            // settled one group at a time: every group's sums at once would not fit the registers
            __asm__ volatile("" : "+v"(k.c[i % NC]), "+v"(k.x[i % NC]));
        }
    }
}

// ---- weights
// A step's code loads of one matrix and its groups' (scale | zero) words.
template <int B, int G>
struct TileW {
    uint4 c[2];
    TileMeta<Lay<B, G>::GSU> m;
};

// Loads of one step of the 16 rows that start at byte offsets co / mo of the
// code and metadata arrays: ol / ml are the lane's offsets for the step, rb8
// the bytes of eight rows.  co and mo of kPastEnd (no such tile), or ol (no
// such step or unit), load zeros; both together wrap to the first lines of
// the array, in range, for a tile whose sums nobody adds.
template <int B, int G>
__device__ __forceinline__ void w_load(TileW<B, G>& w, Rsrc rc, Rsrc rm, uint32_t ol, uint32_t ml, uint32_t rb8,
                                       uint32_t co, uint32_t mo) {
    w.c[0] = bload16<kAuxNt>(rc, ol + co, 0);
    w.c[1] = bload16<kAuxNt>(rc, ol + co + rb8, 0);
    meta_load(w.m, rm, ml + mo);
}

// acc += the step's product with the A operands a.  `tail`: the number of
// groups of this step inside the row (GSU on all but the last step of a
// ragged row).
template <int B, int G>
__device__ __forceinline__ void tile_step(TileW<B, G>& w, const AOps<B, G>& a, const Corr<B, G>& k, f32x4_t& acc,
                                          int tail, int lane) {
    typedef Lay<B, G> Y;
    const uint32_t mv = magic_vgpr();
    const int q = lane >> 4;
    pin4(w.c[0]);
    pin4(w.c[1]);
    arrange<Y::QW != 4, Y::QW == 1>(w.c);
    typedef TileMeta<Y::GSU> Meta;
    if (tail < Y::GSU) {
#pragma unroll
        for (int e = 0; e < Meta::NW; ++e)
            if (meta_first<Y::GSU>(q) + e >= tail)
                w.m.w[e] = 0;
    }
    // the offset and zero-point terms
    if constexpr (Y::GSU == 2) {
        const uint32_t mw = (q & 1) ? w.m.w[1] : w.m.w[0];
        const float sc = h2f(mw & 0xFFFFu);
        acc = mfma4(k.c[0], q < 2 ? sc : sc * h2f(mw >> 16), acc);
    } else {
#pragma unroll
        for (int m = 0; m < Y::GSU / 4; ++m) {
            const float sc = h2f(w.m.w[m] & 0xFFFFu);
            acc = mfma4(k.c[m], sc, acc);
            acc = mfma4(k.x[m], sc * h2f(w.m.w[m] >> 16), acc);
        }
    }
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    if constexpr (Y::HALF) {
        // codes 0..7 or 8..15 of a word as pairs (p, 4 + p) at bits 2 p of both halves
        const uint32_t sel = (q & 1) ? 0x0C030C02u : 0x0C010C00u;
#pragma unroll
        for (int eh = 0; eh < 2; ++eh) {
            float sc[2][4];
            meta_spread(w.m.w[2 * eh], sc[0]);
            meta_spread(w.m.w[2 * eh + 1], sc[1]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // this lane's codes of unit 2 k + eh: groups 4 k + 2 eh and the next
                uint32_t x = word_of(w.c[k >> 1], 2 * (k & 1) + eh), y = x;
                swap16(x, y);
                const uint32_t wd[2] = {__builtin_amdgcn_perm(0u, x, sel), __builtin_amdgcn_perm(0u, y, sel)};
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const uint32_t v = wd[s], v4 = v << 4;
                    const f32x4_t p = mfma16(a[4 * k + 2 * eh + s],
                                             make_uint4(magic(v4, 0x00300030u, mv), magic(v4, 0x00C000C0u, mv),
                                                        magic(v, 0x00300030u, mv), magic(v, 0x00C000C0u, mv)), zero);
                    acc += sc[s][k] * p;
                }
            }
        }
    } else {
        constexpr int NE = Y::GSU == 2 ? 1 : Y::GSU / 4;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            float sc[4];
            if constexpr (Y::GSU == 2) {
                sc[0] = h2f(w.m.w[0] & 0xFFFFu);
                sc[1] = h2f(w.m.w[1] & 0xFFFFu);
            } else {
                meta_spread(w.m.w[e], sc);
            }
#pragma unroll
            for (int k = 0; k < Y::GSU / NE; ++k) {
                const int i = k * NE + e;                  // group of the step
                f32x4_t p = zero;
#pragma unroll
                for (int ww = 0; ww < Y::QW; ++ww) {
                    const uint32_t v = Y::QW == 1   ? word_of(w.c[i >> 2], i & 3)
                                       : Y::QW == 2 ? word_of(w.c[i >> 1], 2 * (i & 1) + ww)
                                                    : word_of(w.c[i & 1], ww);
                    if constexpr (B == 2) {
                        uint32_t x[8];
                        extract_w2(v, x, mv);
                        p = mfma16(a[i * Y::MPG + 2 * ww], make_uint4(x[0], x[1], x[2], x[3]), p);
                        p = mfma16(a[i * Y::MPG + 2 * ww + 1], make_uint4(x[4], x[5], x[6], x[7]), p);
                    } else {
                        uint32_t x[4];
                        extract_w4(v, x, mv);
                        p = mfma16(a[i * Y::MPG + ww], make_uint4(x[0], x[1], x[2], x[3]), p);
                    }
                }
                acc += sc[k] * p;
            }
        }
    }
}

// ---- routed batches (mixture of experts): instance i (token i / xdiv) runs
// expert route[i].  The "blocks" the workgroups walk are the experts that have
// instances, so an expert several tokens share is read once; its instances
// are the operand's 16 rows (an expert of more than 16 counts once per 16).
// Every wave works it out from the ids, one instance per lane.
struct Routed {
    int e;                   // expert of a block
    unsigned long long mask; // its instances
};
__device__ __forceinline__ int route_id(const BatchArgs& b, int n, int lane) {
    int id = lane < n ? b.route[lane] : -1;
    if (lane < n)
        id = id < 0 ? 0 : (id >= b.nexp ? b.nexp - 1 : id);
    return id;
}
__device__ __forceinline__ int route_blocks(const BatchArgs& b, int id) {
    int nv = 0;
    for (int e = 0; e < b.nexp; ++e) nv += (__popcll(__ballot(id == e)) + 15) >> 4;
    return nv;
}
__device__ __forceinline__ Routed route_block(const BatchArgs& b, int id, int l) {
    Routed r{0, 0ull};
    for (int e = 0; e < b.nexp; ++e) {
        const unsigned long long mask = __ballot(id == e);
        const int c = (__popcll(mask) + 15) >> 4;
        if (l < c) {
            r.e = e;
            r.mask = mask;
            for (int i = 0; i < 16 * l; ++i) r.mask &= r.mask - 1;
            break;
        }
        l -= c;
    }
    return r;
}
// The j-th instance of the mask (j < 16); the first where it has fewer.
__device__ __forceinline__ int route_row(unsigned long long mask, int j) {
    int row = __builtin_ctzll(mask);
    for (int i = 0; i < 16 && mask; ++i, mask &= mask - 1)
        if (i == j)
            row = __builtin_ctzll(mask);
    return row;
}

// GU: gate and up of the batch's blocks -> h (MS = 2: a wave takes a tile's
// gate, then its up; MS = 1: one of them, p.mw = 2).  Otherwise the down
// weights of the descriptors on b.h -> b.y (binary16), with p.sk > 1 through
// `scratch`: a counter per workgroup of a slice (kTileCounters words, which
// the gate/up launch before it clears), then the fp32 partials
// [sk][nb][M][N].  Counters and partials are written and read device-coherently
// (the slices run on any XCD) and left at zero.
// PACK (M <= 8, MS = 2): twice the K per register.  The operand of two
// neighbouring steps is one: its rows 0..7 are the tokens at the even step,
// rows 8..15 the tokens at the odd one.  Both steps' weights are multiplied into
// it, into sums of their own, of which the rows of the other step are
// dropped; unit u takes the wave's even (u & 1 = 0) or odd steps of a tile.
// A Qwen3-8B-shaped down half (48 steps) then needs no second slice.
// RT: a routed batch of nb instances of one token each (above); h [nb][f], and
// the linear leaves fp32 [sk][nb][N] in scratch for the combine.
// NSET register sets: NSET - 1 units
// (the SPW steps of one matrix of one tile) are in flight per wave.
template <int B, int G, bool GU, int MS, int SPW, bool PACK, bool RT, int NSET>
__global__ void __launch_bounds__(kTileWaves * 64) tile_kernel(BatchArgs b, int nb, TilePlan p, float* scratch) {
    typedef Lay<B, G> Y;
    static_assert(NSET % MS == 0, "a set holds one matrix or parity");
    static_assert(!PACK || (!GU && MS == 2), "packed steps: linear only");
    constexpr int SK2 = PACK ? 2 : 1;                      // K steps per operand
    constexpr int NM = GU ? 2 : 1;
    const int K = GU ? b.d : b.f, N = GU ? b.f : b.d;
    const int r = GU ? b.r : 0;
    const int tid = threadIdx.x, lane = tid & 63, qt = lane >> 4, jj = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KW = p.kw, TW = p.tw, TG = p.tg, PW = KW * p.mw;    // PW: waves of a tile lane
    const int tw = wave * p.ipw >> 16, pw = wave - tw * PW;
    const int mat = MS == 1 && GU ? pw * p.ikw >> 16 : 0, kw = pw - mat * KW;
    extern __shared__ uint4 smem[];
    // partial sums [2][TG][TW][KW][NM][64], then lora_scale t [2][2][8][64]
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem) + tw * KW * NM * 64 + lane;
    const int tstep = TW * KW * NM * 64;
    float* ts = reinterpret_cast<float*>(reinterpret_cast<f32x4_t*>(smem) + 2 * TG * tstep);
    // the first remainder workgroups (slices) take one tile (step) more
    const int sl = blockIdx.y, wg = blockIdx.x;
    const int sbeg = sl * p.sq + min(sl, p.sr), send = sbeg + p.sq + (sl < p.sr ? 1 : 0);
    const int gs0 = sbeg + kw * SPW * SK2;                 // this wave's first step
    const int rb = K * B / 8, ng = K / G;
    const int tpb = N / 16;
    const int id = RT ? route_id(b, nb, lane) : 0;
    const TileRange own_tiles = RT            ? tile_routed_range(wg, p.wgs, route_blocks(b, id), tpb, TW)
                                : p.wpb > 0 ? tile_range(wg, p.wpb, tpb, p.tq, p.tr, true)
                                            : tile_range(wg, p.wgs, tpb, p.tq, p.tr, false);
    const int t0 = own_tiles.t0, t1 = own_tiles.t1;
    int l = own_tiles.l;
    __shared__ int rows[2][16];                            // RT: instances of a block's operand rows
    KBatchM* kb = kbm();
    uint32_t ol[SPW * SK2];                                // lane's offsets of the code loads
#pragma unroll
    for (int st = 0; st < SPW * SK2; ++st) {
        const int u = (gs0 + st) * 8 + lane_unit<Y::QW == 4>(lane);
        ol[st] = gs0 + st < send && 16 * u < rb ? (uint32_t)((lane & 7) * rb + 16 * u) : kPastEnd;
    }
    const uint32_t ml = (uint32_t)(jj * ng + gs0 * Y::GSU + meta_first<Y::GSU>(qt)) * 4u;
    float* part = scratch + (RT ? 0 : kTileCounters);
    if (!RT && GU && scratch && wg == 0) {
        for (int i = tid; i < kTileCounters; i += p.threads) reinterpret_cast<uint32_t*>(scratch)[i] = 0u;
    }
    if (!RT && !GU && wg == 0 && sl == 0)
        for (int i = tid; i < p.ts; i += p.threads) b.t[i] = 0.0f;
    int buf = 0, fin = 0, par = 0;                         // LDS buffer and adding wave of the next tiles

    for (int seg = t0; seg < t1; ++l) {
        const int tend = (l + 1) * tpb < t1 ? (l + 1) * tpb : t1;
        const int n = (tend - seg + TW - 1) / TW;          // uniform over the workgroup
        const Routed rt = RT ? route_block(b, id, l) : Routed{l, 0ull};
        const int e = rt.e;
        const int M = RT ? min(__popcll(rt.mask), 16) : b.M;     // operand rows in use
        const int own = RT ? route_row(rt.mask, jj) : 0;   // instance of this lane's operand row
        if (RT && wave == 0 && lane < 16)                  // read behind this segment's first barrier
            rows[par][lane] = own;
        const uint32_t cbytes = (uint32_t)N * (uint32_t)rb, mbytes = (uint32_t)N * (uint32_t)ng * 4u;
        const Rsrc rc0 = rsrc(!GU ? kb->lay[e].cd : mat ? kb->lay[e].cu : kb->lay[e].cg, cbytes);
        const Rsrc rm0 = rsrc(!GU ? kb->lay[e].md : mat ? kb->lay[e].mu : kb->lay[e].mg, mbytes);
        const Rsrc rc1 = GU && MS == 2 ? rsrc(kb->lay[e].cu, cbytes) : rc0;
        const Rsrc rm1 = GU && MS == 2 ? rsrc(kb->lay[e].mu, mbytes) : rm0;
        struct Set {
            TileW<B, G> w[SPW];
        };
        // unit u: matrix u % MS of tile u / MS
        auto load = [&](Set& s, int u) {
            const int tile = seg + u / MS * TW + tw;
            const bool real = u < n * MS && tile < tend;
            const uint32_t row = (uint32_t)(tile - l * tpb) * 16u;
#pragma unroll
            for (int st = 0; st < SPW; ++st) {
                const int sp = PACK ? 2 * st + (u & 1) : st;
                w_load<B, G>(s.w[st], MS == 2 && (u & 1) ? rc1 : rc0, MS == 2 && (u & 1) ? rm1 : rm0, ol[sp],
                             ml + 4u * (uint32_t)(sp * Y::GSU), 8u * (uint32_t)rb, real ? row * (uint32_t)rb : kPastEnd,
                             real ? row * (uint32_t)ng * 4u : kPastEnd);
            }
        };
        // This block's activations, ahead of the first weights: behind them they wait in the memory's queues
        // (one Qwen3-8B-shaped down half: 14.0 us this way, 17.8 the other).
        AOps<B, G> a[SPW];
        {
            const int la = fresh(lane);
            const Rsrc rx = RT ? rsrc(GU ? b.x : b.h, (uint32_t)(GU ? nb / b.xdiv : nb) * (uint32_t)K * 2u)
                               : rsrc((GU ? b.x : b.h) + (long)l * M * K, (uint32_t)M * (uint32_t)K * 2u);
#pragma unroll
            for (int st = 0; st < SPW; ++st) {
                const int gs = PACK ? gs0 + 2 * st + ((la >> 3) & 1) : gs0 + st;
                if constexpr (RT)
                    act_load<B, G>(a[st], rx, gs, GU ? own / b.xdiv : own, nb, K, gs < send && (la & 15) < M, la);
                else
                    act_load<B, G>(a[st], rx, gs, PACK ? la & 7 : la & 15, M, K, gs < send, la);
            }
        }
        // LoRA-B of the tile this wave adds in the group of TG tiles from i on:
        // r/4 halves (ranks q r/4 ..) of the lane's row of B_gate and B_up
        uint4 lb[NM];
        auto lora_load = [&](int i) {
            if constexpr (GU) {
                const int k = pw >= fin ? pw - fin : pw - fin + PW;
                const int tile = seg + (i + k) * TW + tw;
                const bool real = r > 0 && k < TG && i + k < n && tile < tend;
                const uint32_t bytes = (uint32_t)N * (uint32_t)r * 2u;
                const int la = fresh(lane);
                const uint32_t o = real ? (uint32_t)((tile - l * tpb) * 16 * r + (la & 15) * r + (la >> 4) * (r / 4)) * 2u
                                        : kPastEnd;
                lb[0] = bload16<0>(rsrc(kb->lay[e].Bg, bytes), o, 0);
                lb[1] = bload16<0>(rsrc(kb->lay[e].Bu, bytes), o, 0);
            }
        };
        // ts[m][u][16 q + j] = lora_scale t[token j][rank q r/4 + u], the slices of d in order; read behind
        // this segment's first barrier.
        const int lg = r == 8 ? 1 : r == 16 ? 2 : 3;       // r / 4 = 2^lg
        const int nts = GU && r > 0 ? 2 * (r / 4) * 64 : 0;
        auto t_load = [&](int i, float (&v)[kLoraSlices]) {
            const int j = i & 15, q = (i >> 4) & 3, m = i >> (6 + lg), u = (i >> 6) - (m << lg);
            const long row = RT ? own : (long)l * M + (j < M ? j : 0);     // i & 15 = lane & 15
            const float* tc = b.t + row * 2 * r + m * r + q * (r / 4) + u;
#pragma unroll
            for (int sl = 0; sl < kLoraSlices; ++sl)
                v[sl] = tc[(long)(sl < p.ts ? sl : 0) * nb * (RT ? 1 : M) * 2 * r];
        };
        auto t_store = [&](int i, const float (&v)[kLoraSlices]) {
            const int j = i & 15, m = i >> (6 + lg), u = (i >> 6) - (m << lg);
            float t = v[0];
#pragma unroll
            for (int sl = 1; sl < kLoraSlices; ++sl)
                if (sl < p.ts)
                    t += v[sl];
            ts[par * 1024 + (m * 8 + u) * 64 + (i & 63)] = j < M ? kb->lay[e].lora_scale * t : 0.0f;
        };
        float tv[2][kLoraSlices];
        if (nts > 0) {
            const int i = fresh(tid);
            t_load(i < nts ? i : 0, tv[0]);
            t_load(i + p.threads < nts ? i + p.threads : 0, tv[1]);
        }
        Set S[NSET];
#pragma unroll
        for (int s = 0; s < NSET - 1; ++s) load(S[s], s);
        Corr<B, G> cr[SPW];
#pragma unroll
        for (int st = 0; st < SPW; ++st) {
            act_mask<B, G>(a[st], PACK ? gs0 + 2 * st + ((lane >> 3) & 1) : gs0 + st, K, lane);
            act_convert<B, G>(a[st]);
            group_sums<B, G>(a[st], cr[st], lane);
        }
        if (nts > 0) {
            const int i = fresh(tid);
            if (i < nts) t_store(i, tv[0]);
            if (i + p.threads < nts) t_store(i + p.threads, tv[1]);
            for (int k = i + 2 * p.threads; k < nts; k += p.threads) {
                t_load(k, tv[0]);
                t_store(k, tv[0]);
            }
        }
        lora_load(0);
        int g = 0;                                         // tile within its group
        // Partial sums of tiles i - g .. i meet: wave fin + k adds those of the
        // group's k-th tile, with LoRA-B and SiLU(G) * U for gate/up.
        auto finish = [&](int i) {
            lds_barrier();
            const int k = pw >= fin ? pw - fin : pw - fin + PW;
            const int tile = seg + (i - g + k) * TW + tw;
            if (k <= g && tile < tend) {
                const f32x4_t* rd = red + (buf * TG + k) * tstep;
                f32x4_t acc[NM];
#pragma unroll
                for (int m = 0; m < NM; ++m) acc[m] = rd[m * 64];
#pragma unroll 4
                for (int w = 1; w < KW; ++w) {
#pragma unroll
                    for (int m = 0; m < NM; ++m) acc[m] += rd[(w * NM + m) * 64];
                }
#pragma unroll
                for (int m = 0; m < NM; ++m) acc[m] *= kTileUnscale;
                if constexpr (GU) {
                    if (r > 0) {
#pragma unroll
                        for (int m = 0; m < NM; ++m) {
                            const uint32_t w[4] = {lb[m].x, lb[m].y, lb[m].z, lb[m].w};
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                if ((u == 2 && r < 16) || (u == 4 && r < 32))
                                    break;
                                acc[m] = mfma4(ts[par * 1024 + (m * 8 + u) * 64 + lane],
                                               h2f((w[u >> 1] >> (16 * (u & 1))) & 0xFFFFu), acc[m]);
                            }
                        }
                    }
                }
                const int la = fresh(lane), o = (tile - l * tpb) * 16 + (la & 15);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int tok = 4 * (la >> 4) + v;
                    if (tok < M) {
                        const long at = (RT ? (long)rows[par][tok] : (long)l * M + tok) * N + o;
                        if constexpr (GU) {
                            const float gv = acc[0][v];
                            b.h[at] = (uint16_t)f2h(gv / (1.0f + __expf(-gv)) * acc[1][v]);
                        } else if (RT) {
                            part[(long)sl * nb * N + at] = acc[0][v];
                        } else if (p.sk > 1) {
                            __hip_atomic_store(part + (long)sl * nb * M * N + at, acc[0][v], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                        } else {
                            b.y[at] = (uint16_t)f2h(acc[0][v]);
                        }
                    }
                }
            }
            buf ^= 1;
            fin += g + 1;
            if (fin >= PW) fin -= PW;                      // g + 1 <= TG <= PW
            g = 0;
            lora_load(i + 1);
        };
        f32x4_t even = {0.f, 0.f, 0.f, 0.f};               // PACK: the even steps' sums
        auto run = [&](Set& s, int u) {
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < SPW; ++st)
                tile_step<B, G>(s.w[st], a[st], cr[st], acc, ng - (gs0 + (PACK ? 2 * st + (u & 1) : st)) * Y::GSU, lane);
            if constexpr (PACK) {
                if ((u & 1) == 0) {
                    even = acc;
                    return;
                }
                // rows 8..15 of the odd steps' sums (lanes 32..63) join rows 0..7 of the even ones'
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    uint32_t x = __float_as_uint(acc[v]), y = x;
                    swap32(x, y);
                    acc[v] = even[v] + __uint_as_float(y);
                }
            }
            red[(buf * TG + g) * tstep + (kw * NM + (GU && MS == 2 ? u & 1 : mat)) * 64] = acc;
            if (MS == 1 || (u & 1)) {
                const int i = u / MS;
                if (g + 1 == TG || i + 1 == n)
                    finish(i);
                else
                    ++g;
            }
        };
        for (int u = 0; u < n * MS; u += NSET) {
#pragma unroll
            for (int s = 0; s < NSET; ++s) {
                load(S[(s + NSET - 1) % NSET], u + s + NSET - 1);
                if (u + s < n * MS)
                    run(S[s], u + s);
            }
        }
        seg = tend;
        par ^= 1;
    }
    if constexpr (!GU && !RT) {
        const int M = b.M;
        if (p.sk > 1) {
            // every partial of this workgroup is out, then the range's counter: the last slice adds them all
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            uint32_t* last = reinterpret_cast<uint32_t*>(smem);
            if (tid == 0)
                *last = __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(scratch) + wg, 1u, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (*last != (uint32_t)p.sk - 1u)
                return;
            // the scratch goes back to zeros: it may lie where another call's hand-off words are expected
            if (tid == 0)
                reinterpret_cast<uint32_t*>(scratch)[wg] = 0u;
            const uint32_t slice = (uint32_t)nb * (uint32_t)M * (uint32_t)N * 4u;
            const Rsrc rp = rsrc(part, slice * (uint32_t)p.sk);
            const int tok = lane >> 2;                     // four rows of one token per lane
            for (int tile = t0 + wave; tile < t1; tile += p.threads >> 6) {
                const int bl = nb == 1 ? 0 : (unsigned)tile / (unsigned)tpb;
                if (tok < M) {
                    const uint32_t at = (uint32_t)(bl * M + tok) * (uint32_t)N + (uint32_t)(tile - bl * tpb) * 16u +
                                        4u * (uint32_t)(lane & 3);
                    float y[4] = {0.f, 0.f, 0.f, 0.f};
                    for (int s = 0; s < p.sk; ++s) {
                        const uint4 v = bload16<kAuxDevice>(rp, at * 4u + (uint32_t)s * slice, 0);
                        *reinterpret_cast<uint4*>(part + at + (uint32_t)s * (slice / 4u)) = make_uint4(0u, 0u, 0u, 0u);
                        y[0] += __uint_as_float(v.x);
                        y[1] += __uint_as_float(v.y);
                        y[2] += __uint_as_float(v.z);
                        y[3] += __uint_as_float(v.w);
                    }
                    *reinterpret_cast<uint2*>(b.y + at) =
                        make_uint2(f2h(y[0]) | (f2h(y[1]) << 16), f2h(y[2]) | (f2h(y[3]) << 16));
                }
            }
        }
    }
}


// ---- LoRA-A: t = [A_g; A_u] x of every block (Sec. 3.1 Eq. (1), Sec. 4.2).
// A workgroup multiplies 16 rows of [A_g; A_u] (those past r are A_u's) by the
// block's tokens over one of S slices of d; its four waves take a share of
// it each, in steps of 32 whose loads go out four at a time, and add their
// sums in wave order through LDS into t [S][nb][M][2r] fp32; the gate/up
// launch adds the slices in order.  The launch is one trip to memory, so it
// is spread over as many compute units as there is room for partials: one
// Qwen3-8B-shaped block at M = 8 takes 4.5 us with four slices, 8.0 with one.
// RT: a routed batch of nb instances, block l its l-th expert; t [S][nb][2r].
template <bool RT>
__global__ void __launch_bounds__(256) tile_lora_kernel(BatchArgs b, int nb, int S) {
    __shared__ f32x4_t red[4][64];
    const int d = b.d, r = b.r;
    const int s = blockIdx.z, tile = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4;
    const int id = RT ? route_id(b, nb, lane) : 0;
    const Routed rt = RT ? route_block(b, id, blockIdx.y) : Routed{(int)blockIdx.y, 0ull};
    if (RT && !rt.mask)
        return;                                            // fewer experts than instances
    const int l = rt.e, M = RT ? min(__popcll(rt.mask), 16) : b.M;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = tile * 16 + (lane & 15);                 // this lane's row of [A_g; A_u]
    const int all = d / 32, w = 4 * s + wave, s0 = w * all / (4 * S), n = (w + 1) * all / (4 * S) - s0;
    const uint16_t* ar = (c < r ? kbm()->lay[l].Ag + (long)c * d : kbm()->lay[l].Au + (long)(c - r) * d) + s0 * 32 + 8 * q;
    const int j = (lane & 15) < M ? (lane & 15) : 0;       // rows past M: token 0, dropped
    const uint16_t* xr = b.x + (RT ? (long)(route_row(rt.mask, j) / b.xdiv) : (long)l * M + j) * d + s0 * 32 + 8 * q;
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int KC = 4;
    for (int i = 0; i < n; i += KC) {
        uint4 av[KC], xv[KC];
#pragma unroll
        for (int u = 0; u < KC; ++u) {
            const int k = 32 * (i + u < n ? i + u : n - 1);
            av[u] = *reinterpret_cast<const uint4*>(ar + k);
            xv[u] = *reinterpret_cast<const uint4*>(xr + k);
        }
#pragma unroll
        for (int u = 0; u < KC; ++u)
            if (i + u < n)
                acc = mfma16(xv[u], av[u], acc);
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
        const f32x4_t t = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (4 * q + v < M)
                b.t[(RT ? (long)s * nb + route_row(rt.mask, 4 * q + v) : ((long)s * nb + l) * M + 4 * q + v) * 2 * r + c] = t[v];
    }
}

}  // namespace

bool tile_gateup_supported(int M, int d, int f, int g, int bits, int r, int nb) {
    TilePlan p;
    return plan_gateup(M, d, f, g, bits, r, nb, false, device_cus(), p);
}

int tile_linear_slices(int M, int n, int k, int g, int bits, int nb) {
    TilePlan p;
    return plan_linear(M, n, k, g, bits, nb, false, device_cus(), p) && (p.sk == 1 || p.wgs <= kTileCounters) ? p.sk : 0;
}
size_t tile_scratch_bytes(int sk, int nb, int M, int n) {
    return sk > 1 ? (size_t)kTileCounters * 4 + (size_t)sk * nb * M * n * 4 : 0;
}

template <typename KERNEL>
static hipError_t tile_run(KERNEL k, const BatchArgs& b, int nb, const TilePlan& p, float* scratch, hipStream_t st) {
    hipError_t e = set_lds(k, p.lds);
    if (e != hipSuccess)
        return e;
    k<<<dim3((unsigned)p.wgs, (unsigned)p.sk), (unsigned)p.threads, p.lds, st>>>(b, nb, p, scratch);
    return hipGetLastError();
}

hipError_t launch_lora_a_tile(const BatchArgs& b, int nb, int slices, hipStream_t st) {
    if (slices < 1 || slices > kLoraSlices || b.M < 1 || b.M > 16 || nb < 1 || nb > kBatchMax || b.d % 64 != 0 || (b.r != 8 && b.r != 16 && b.r != 32))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)(2 * b.r / 16), (unsigned)nb, (unsigned)slices);
    if (b.route)
        tile_lora_kernel<true><<<grid, 256, 0, st>>>(b, nb, slices);
    else
        tile_lora_kernel<false><<<grid, 256, 0, st>>>(b, nb, slices);
    return hipGetLastError();
}

// Register sets of the gate/up half where gate and up have waves of their own:
// 2-bit groups of 32 hold sixteen groups' (scale | zero) words a step, and a
// fourth set spills (1 to 4 registers; 36 blocks of d = 2560, f = 9728 at 5
// tokens 305.5 us with four sets, 302 with three; 4 at 16 66.0 and 64.1).
// In turn, gate and up take an even number: four sets, of which only the
// routed instance of those groups spills (3 registers).
constexpr int gu_sets(int bits, int g) { return bits == 2 && g == 32 ? 3 : 4; }

hipError_t launch_gateup_tile(const BatchArgs& b, int nb, int slices, float* scratch, hipStream_t st) {
    TilePlan p;
    if (!plan_gateup(b.M, b.d, b.f, b.gg, b.bg, b.r, nb, b.route != nullptr, device_cus(), p))
        return hipErrorInvalidValue;
    p.ts = slices;
#define QMLP_TGU_R(B_, G_, R_)                                                            \
    if (b.bg == B_ && b.gg == G_ && (b.route != nullptr) == R_)                           \
        return p.mw == 2 ? tile_run(tile_kernel<B_, G_, true, 1, 1, false, R_, gu_sets(B_, G_)>, b, nb, p, scratch, st) \
                         : tile_run(tile_kernel<B_, G_, true, 2, 1, false, R_, 4>, b, nb, p, scratch, st);
#define QMLP_TGU(B_, G_) QMLP_TGU_R(B_, G_, false) QMLP_TGU_R(B_, G_, true)
    QMLP_TGU(2, 128) QMLP_TGU(2, 64) QMLP_TGU(2, 32) QMLP_TGU(4, 128) QMLP_TGU(4, 64) QMLP_TGU(4, 32)
    return hipErrorInvalidValue;
}

hipError_t launch_linear_tile(const BatchArgs& b, int nb, int clear_t, float* scratch, hipStream_t st) {
    TilePlan p;
    // a routed batch: up to 16 operand rows, partials always
    if (!plan_linear(b.route ? 16 : b.M, b.d, b.f, b.gd, b.bd, nb, b.route != nullptr, device_cus(), p) || ((p.sk > 1 || b.route) && !scratch))
        return hipErrorInvalidValue;
    p.ts = clear_t;
#define QMLP_TLN(B_, G_, S_)                                                              \
    if (b.bd == B_ && b.gd == G_)                                                         \
        return b.route ? tile_run(tile_kernel<B_, G_, false, 1, S_, false, true, 3>, b, nb, p, scratch, st) \
               : p.pack ? tile_run(tile_kernel<B_, G_, false, 2, S_, true, false, 2>, b, nb, p, scratch, st) \
                        : tile_run(tile_kernel<B_, G_, false, 1, S_, false, false, 3>, b, nb, p, scratch, st);
    QMLP_TLN(4, 128, 2) QMLP_TLN(4, 64, 2) QMLP_TLN(4, 32, 1) QMLP_TLN(2, 128, 1) QMLP_TLN(2, 64, 1)
    return hipErrorInvalidValue;
}

}  // namespace qmlp
