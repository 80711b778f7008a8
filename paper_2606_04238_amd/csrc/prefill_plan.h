// How a prefill chunk (prefill.hip) is split: the tile of the gate/up kernel,
// the token tile and the slices of f of the down kernel.  Plain host C++ over
// sizes and compute units, so that the rules can be checked without a device.
#pragma once

#include <stddef.h>

namespace qmlp {

constexpr int PF_BK = 64;              // input elements per step
constexpr int kDownSlicesMax = 8;

// Token tile of the down kernel: 256 tokens (8 waves; every
// dequantized weight serves 256 tokens) where M allows, else 128 (4 waves).
inline int prefill_bm(int M) { return M % 256 == 0 ? 256 : 128; }

// Tokens and columns of h of a gate/up workgroup.
struct PrefillTile {
    int bm, hc;
};
// Three tiles: 256 tokens x 128 columns of h and 256 x 64 (one workgroup per
// compute unit), 128 x 64 (two; the only one for an odd number of 128-token
// tiles).  A larger tile moves less through LDS per matrix instruction but
// leaves more of the chip idle when there are few, so the one whose rounds
// over the chip take the least time is used; a round measured 1 : 0.62 :
// 0.77 (0.5 where the small tiles get a compute unit each).  4B shape
// (d = 2560, f = 9728), whole chunk, us, in that order: M = 256 111, 81,
// 93; M = 512 139, 151, 151; M = 1024 258, 241, 248.  20B-class, M = 512:
// 358, 383, 433; M = 256: 269, 214, 240.
inline PrefillTile prefill_gateup_tile(int M, int f, int cus) {
    const auto rounds = [&](int bm, int hc, int per_cu) {
        return (double)(((long)(M / bm) * (f / hc) + per_cu * cus - 1) / (per_cu * cus));
    };
    const double c64 = M % 256 == 0 ? 0.62 * rounds(256, 64, 1) : 1e30;
    const double c128 = M % 256 == 0 && f % 128 == 0 ? rounds(256, 128, 1) : 1e30;
    const double csmall = (long)(M / 128) * (f / 64) <= cus ? 0.5 : 0.77 * rounds(128, 64, 2);
    const int hc = c128 <= c64 && c128 <= csmall ? 128 : 64;
    return {hc == 128 || c64 <= csmall ? 256 : 128, hc};
}

// The most slices of f a chunk's down half may take (the workspace is sized
// for them): doubled while under 512 tiles, slices of whole 64-wide steps.
inline int prefill_down_slices_most(int M, int d, int f) {
    const long tiles = (long)(M / prefill_bm(M)) * (d / 128);
    int S = 1;
    while (S < kDownSlicesMax && tiles * S < 512 && f % (2 * S * PF_BK) == 0) S *= 2;
    return S;
}

// The slices it takes: as many as keep (token tile x row tile x slice) within
// one round over the compute units (of 128-token workgroups two fit one, and
// a quarter more than that still pays: M = 640 of the 8B shape 312 us with 640
// workgroups, 316 with 320).  A second round costs more than the finer
// slices save, and every slice writes and re-reads its partials: 4B shape,
// M = 512, 4 slices (160 workgroups) 132 us per chunk, 8 (320) 138; M = 1024, 2
// (160) 242, 8 260; M = 2048, 1 (160) 390, 4 398; 20B-class, M = 256, 4 (192)
// 256, 8 269, M = 512, 2 (192) and 8 363.
inline int prefill_down_slices(int M, int d, int f, int cus) {
    const long tiles = (long)(M / prefill_bm(M)) * (d / 128);
    int S = prefill_down_slices_most(M, d, f);
    while (S > 1 && 2 * tiles * S > (prefill_bm(M) == 128 ? 5 : 2) * (long)cus) S /= 2;
    return S;
}

}  // namespace qmlp
