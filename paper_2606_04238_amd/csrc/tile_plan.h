// How the tile kernels (decode_tile.hip) split a call: waves, tiles,
// workgroups, slices and LDS of a launch, and which shapes do not fit.  Plain
// host C++ over sizes and the number of compute units, so that the rules can
// be checked without a device.
#pragma once

#include <stddef.h>

namespace qmlp {

constexpr int kTileBatch = 40;                    // blocks of a batch, instances of a routed one
constexpr int kTileWaves = 12;                    // waves of a workgroup, 168 registers each
constexpr size_t kTileLds = 159 * 1024;           // beside the routed batch's row table
constexpr int kTileCounters = 256;                // words at the start of the scratch

struct TilePlan {
    int kw, tw;              // waves along K, tiles side by side
    int mw;                  // gate/up: 2 where gate and up have waves of their own, else 1
    int tg;                  // tiles of a tile lane per barrier
    int sk, ns;              // K slices, steps of a row
    int wgs;                 // workgroups per K slice
    int wpb;                 // workgroups per block, 0: every workgroup its share of the whole batch
    int tq, tr;              // tiles (of a block, of the batch) over those workgroups: quotient, remainder
    int sq, sr;              // steps of a row over slices
    int ipw, ikw;            // 2^16 / waves of a tile lane and / kw, rounded up (waves are below 16)
    int pack;                // packed steps
    int ts;                  // gate/up: slices of d in t; linear: floats of t to clear
    int threads;
    size_t lds;
};

// Tiles side by side: as many as the workgroup's waves allow, but no more than
// leave every compute unit a workgroup.
inline int tile_tw(long tiles, int pw, int sk, int cus) {
    const long most = kTileWaves / pw, spread = tiles * sk / cus;
    return (int)(spread < 1 ? 1 : spread < most ? spread : most);
}

// Workgroups of a launch: one per compute unit over all slices, no more than
// there are groups of TW tiles.
inline int tile_wgs(long tiles, int tw, int sk, int cus) {
    const long most = (tiles + tw - 1) / tw, per = cus / sk > 0 ? cus / sk : 1;
    return (int)(most < per ? most : per);
}

// The kernel's divisions, done here.
inline void tile_shares(TilePlan& p, long tiles) {
    p.tq = (int)(tiles / p.wgs);
    p.tr = (int)(tiles % p.wgs);
    p.sq = p.ns / p.sk;
    p.sr = p.ns % p.sk;
    p.ipw = 65536 / (p.kw * p.mw) + 1;
    p.ikw = 65536 / p.kw + 1;
}

// Tiles per barrier: up to four (a wave of its own adds each), as LDS allows;
// false where not even one fits.
inline bool tile_group(TilePlan& p, int nm, size_t more) {
    p.tg = p.kw * p.mw < 4 ? p.kw * p.mw : 4;
    for (;; --p.tg) {
        p.lds = (size_t)2 * p.tg * p.tw * p.kw * nm * 1024 + more;
        if (p.lds <= kTileLds)
            return true;
        if (p.tg == 1)
            return false;
    }
}

// Workgroups of their own for each block of a batch, or an even share of the
// whole batch for every workgroup?  A workgroup that crosses into another block
// stages new activations with no weights in flight, which measured 7 us, about
// the time of kCross tiles; whole workgroups per block leave some compute units
// without work or the largest share a tile longer.  Own workgroups against an
// even share: 12 blocks of d = 2048, f = 6144 at M = 16 63 against 71 us, 20 of
// d = f = 2880 69 against 74, 36 Qwen3-4B-shaped ones 227 against 230.
// nb blocks of tpb tiles, tw side by side, over wgs workgroups: the workgroups
// of each block, 0 for even shares.
constexpr int tile_own(int wgs, int nb, int tpb, int tw) {
    constexpr int kCross = 5;
    const int per = wgs / nb < (tpb + tw - 1) / tw ? wgs / nb : (tpb + tw - 1) / tw;
    const int shared = (int)(((long)nb * tpb + wgs - 1) / wgs) + kCross * tw;
    return nb > 1 && per >= 1 && (tpb + per - 1) / per <= shared ? per : 0;
}
inline void tile_blocks(TilePlan& p, int nb, int tpb, int cus) {
    p.wpb = tile_own(cus / p.sk, nb, tpb, p.tw);
    if (p.wpb > 0) {
        p.wgs = p.wpb * nb;
        p.tq = tpb / p.wpb;
        p.tr = tpb % p.wpb;
    }
}

// The tiles [t0, t1) of workgroup wg, the first of them of block l.
struct TileRange {
    int l, t0, t1;
};
constexpr TileRange tile_range(int wg, int wgs, int tpb, int tq, int tr, bool own) {
    // workgroups 0 .. tr - 1 (of a block's own ones, or of all) take a tile more
    const int l = own ? (int)((unsigned)wg / (unsigned)wgs) : 0;
    const int i = own ? wg - l * wgs : wg;
    const int t0 = l * tpb + i * tq + (i < tr ? i : tr);
    return {own ? l : (int)((unsigned)t0 / (unsigned)tpb), t0, t0 + tq + (i < tr ? 1 : 0)};
}
// ... of a routed batch, whose blocks are the nv experts that have instances:
// known in the kernel only, so the launch has workgroups for every compute
// unit and the kernel applies the rule above (workgroups past the experts'
// own stay idle).  With the shares made on the host for the instances (40 of
// them on 240 workgroups) 20B-class layers at 8, 9 and 10 tokens took 85-89,
// 88-95 and 89-99 us over four routings, this way 78-83, 83-85 and 84-89; even
// shares throughout 94 against 87 where the 240 happened to divide the experts.
constexpr TileRange tile_routed_range(int wg, int wgs, int nv, int tpb, int tw) {
    const int own = tile_own(wgs, nv, tpb, tw);
    if (own > 0 && wg >= own * nv)
        return {0, 0, 0};
    const int over = own > 0 ? own : wgs, tiles = own > 0 ? tpb : nv * tpb;
    const int tq = (int)((unsigned)tiles / (unsigned)over);
    return tile_range(wg, over, tpb, tq, tiles - tq * over, own > 0);
}

// Gate/up: K = d.  Gate and up take waves of their own while both fit in one
// workgroup (twice the waves share the stream of a short row), else every
// wave takes a tile's gate, then its up.  Rows past kTileWaves steps do not
// fit: false.
inline bool plan_gateup(int M, int d, int f, int g, int bits, int r, int nb, bool routed, int cus, TilePlan& p) {
    if (cus <= 0 || M < 1 || M > 16 || nb < 1 || nb > kTileBatch || d % 64 != 0 || f % 16 != 0 || d % g != 0 ||
        (bits != 2 && bits != 4) || (r != 0 && r != 8 && r != 16 && r != 32) ||
        (long)f * d * bits / 8 >= (1l << 31) || (long)f * (d / g) * 4 >= (1l << 31))
        return false;
    const int cps = 1024 / bits;
    p.ns = (d + cps - 1) / cps;
    p.sk = 1;
    p.pack = 0;
    p.kw = p.ns;
    p.mw = 2 * p.kw <= kTileWaves ? 2 : 1;
    if (p.kw > kTileWaves)
        return false;
    p.tw = tile_tw((long)nb * (f / 16), p.kw * p.mw, 1, cus);
    p.threads = p.tw * p.kw * p.mw * 64;
    p.wgs = tile_wgs((long)nb * (f / 16), p.tw, 1, cus);
    p.wpb = 0;
    tile_shares(p, (long)nb * (f / 16));
    if (!routed)
        tile_blocks(p, nb, f / 16, cus);
    return tile_group(p, 2, r > 0 ? 8192 : 0);
}

// 4-bit groups of 32 hold one step per wave (two spill).
inline int linear_spw(int g, int bits) { return bits == 4 && g != 32 ? 2 : 1; }

// Any linear [n][k]: as few slices of k as fit the workgroup's registers, with
// packed steps where that saves slices, and for rows past sixteen steps where
// a workgroup has one tile at most: then half the waves stage and meet, and
// nothing streams that they could share (us, unpacked and packed, one matrix
// of 2048 rows in groups of 128: k = 5120 at 2, 4 and 8 tokens 7.7, 8.0, 8.8
// and 6.6, 7.2, 7.9, k = 4608 at 2 7.2 and 6.8; past a tile per compute unit
// both the same or the stream counts, and rows of sixteen steps and fewer
// start as fast either way).
inline bool plan_linear(int M, int n, int k, int g, int bits, int nb, bool routed, int cus, TilePlan& p) {
    if (cus <= 0 || M < 1 || M > 16 || nb < 1 || nb > kTileBatch || k % 64 != 0 || n % 16 != 0 || k % g != 0 ||
        (bits != 2 && bits != 4) || (bits == 2 && g == 32) || (long)n * k * bits / 8 >= (1l << 31) ||
        (long)n * (k / g) * 4 >= (1l << 31))
        return false;
    const int cps = 1024 / bits, spw = linear_spw(g, bits);
    p.ns = (k + cps - 1) / cps;
    const bool few = spw == 2 && p.ns > 8 * spw && (long)nb * (n / 16) <= cus;
    p.pack = M <= 8 && (p.ns > kTileWaves * spw || few) ? 1 : 0;
    const int per = spw << p.pack;                         // steps per wave
    p.sk = (p.ns + kTileWaves * per - 1) / (kTileWaves * per);
    if ((long)p.sk * nb * M * n * 4 >= (1l << 31) || p.sk > cus)
        return false;
    p.kw = ((p.ns + p.sk - 1) / p.sk + per - 1) / per;
    p.mw = 1;
    p.tw = tile_tw((long)nb * (n / 16), p.kw, p.sk, cus);
    p.threads = p.tw * p.kw * 64;
    p.wgs = tile_wgs((long)nb * (n / 16), p.tw, p.sk, cus);
    p.wpb = 0;
    tile_shares(p, (long)nb * (n / 16));
    if (!routed)
        tile_blocks(p, nb, n / 16, cus);
    return tile_group(p, 1, 0);
}

}  // namespace qmlp
