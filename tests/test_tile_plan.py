"""The split of the tile kernels' launches (csrc/tile_plan.h, host C++ over
sizes and compute units), compiled here with g++ and checked without a GPU:
every tile of every block belongs to one workgroup and every step of a row to
one wave, LDS and the slices' counters suffice, and the chip is used."""
import ctypes
import shutil

import pytest

from qmlp_testutil import host_library

FIELDS = ("kw", "tw", "mw", "tg", "sk", "ns", "wgs", "wpb", "tq", "tr", "sq", "sr", "ipw", "ikw", "pack",
          "threads", "lds")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

SRC = """
#include "tile_plan.h"
using namespace qmlp;
static int put(const TilePlan& p, long* o) {
    const long v[] = {%s};
    for (unsigned i = 0; i < sizeof v / sizeof *v; ++i) o[i] = v[i];
    return 1;
}
extern "C" int gateup(int M, int d, int f, int g, int bits, int r, int nb, int routed, int cus, long* o) {
    TilePlan p{};
    return plan_gateup(M, d, f, g, bits, r, nb, routed != 0, cus, p) ? put(p, o) : 0;
}
extern "C" int linear(int M, int n, int k, int g, int bits, int nb, int routed, int cus, long* o) {
    TilePlan p{};
    return plan_linear(M, n, k, g, bits, nb, routed != 0, cus, p) ? put(p, o) : 0;
}
extern "C" void range(int wg, int wpb, int wgs, int tpb, int tq, int tr, long* o) {
    const TileRange t = wpb > 0 ? tile_range(wg, wpb, tpb, tq, tr, true) : tile_range(wg, wgs, tpb, tq, tr, false);
    o[0] = t.l; o[1] = t.t0; o[2] = t.t1;
}
extern "C" void routed_range(int wg, int wgs, int nv, int tpb, int tw, long* o) {
    const TileRange t = tile_routed_range(wg, wgs, nv, tpb, tw);
    o[0] = t.l; o[1] = t.t0; o[2] = t.t1;
}
""" % ", ".join("(long)p." + f for f in FIELDS)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = host_library(SRC, tmp_path_factory.mktemp("plan"))

    def call(which, *args, cus=256):
        out = (ctypes.c_long * len(FIELDS))()
        ok = getattr(lib, which)(*[ctypes.c_int(a) for a in args], ctypes.c_int(cus), out)
        return dict(zip(FIELDS, out)) if ok else None

    def ranges(which, wgs, *args):
        o = (ctypes.c_long * 3)()
        for wg in range(wgs):
            getattr(lib, which)(*[ctypes.c_int(a) for a in (wg,) + args], o)
            yield tuple(o)
    call.ranges = ranges
    return call


def _cover(ranges, tiles, tpb):
    """The ranges are the tiles 0 .. tiles - 1 in order, each with its first tile's block; the longest."""
    at = most = 0
    for l, t0, t1 in ranges:
        if t0 < t1:
            assert t0 == at and l == t0 // tpb
            at, most = t1, max(most, t1 - t0)
    assert at == tiles
    return most


def _check(plan, p, tiles, nb, nm, M, n, routed=False, cus=256):
    waves = p["kw"] * p["mw"] * p["tw"]
    assert p["threads"] == 64 * waves <= 64 * 12
    assert 1 <= p["tg"] <= min(4, p["kw"] * p["mw"])                # a wave of its own adds each tile of a group
    assert 2 * p["tg"] * p["tw"] * p["kw"] * nm * 1024 <= p["lds"] <= 159 * 1024
    assert 1 <= p["wgs"] and p["wgs"] * p["sk"] <= max(cus, p["sk"])
    for w in range(waves):                                          # the kernel's divisions
        assert w * p["ipw"] >> 16 == w // (p["kw"] * p["mw"])
        assert w * p["ikw"] >> 16 == w // p["kw"]
    # tiles: quotient and remainder over a block's workgroups or all of them
    if not routed:
        assert not p["wpb"] or p["wpb"] * nb == p["wgs"]
        _cover(plan.ranges("range", p["wgs"], p["wpb"], p["wgs"], tiles, p["tq"], p["tr"]), nb * tiles, tiles)
    # steps: the slices' shares, each within its waves' operands
    assert p["sq"] * p["sk"] + p["sr"] == p["ns"] and 0 <= p["sr"] < p["sk"]
    if p["sk"] > 1:
        assert p["wgs"] <= 256 and p["sk"] * nb * M * n * 4 < 1 << 31
    if routed:
        assert p["wpb"] == 0


@pytest.mark.parametrize("bits,g", [(2, 32), (2, 64), (2, 128), (4, 32), (4, 64), (4, 128)])
@pytest.mark.parametrize("nb", [1, 2, 7, 20, 36, 40])
def test_plans_cover_every_tile_and_step(plan, bits, g, nb):
    for M in (1, 2, 8, 9, 16):
        for k in (g * ((64 + g - 1) // g), 576 // g * g or g, 1344 // g * g, 2560, 2944, 3072, 4096, 6144, 6272,
                  12288, 17408, 28672):
            if k % 64:
                continue
            for n in (64, 448, 2560, 12288):
                for routed in (False, True):
                    p = plan("gateup", M, k, n, g, bits, 16, nb, int(routed))
                    assert (p is None) == ((k + 1024 // bits - 1) // (1024 // bits) > 12)
                    if p:
                        assert p["ns"] == p["kw"] and p["sk"] == 1
                        _check(plan, p, n // 16, nb, 2, M, n, routed)
                    if bits == 2 and g == 32:
                        continue
                    p = plan("linear", M, n, k, g, bits, nb, int(routed))
                    assert p is not None
                    per = (2 if bits == 4 and g != 32 else 1) << p["pack"]
                    assert p["kw"] * per >= p["sq"] + (p["sr"] > 0) and p["kw"] <= 12
                    assert not p["pack"] or M <= 8
                    _check(plan, p, n // 16, nb, 1, M, n, routed)


@pytest.mark.parametrize("n", [1, 2, 7, 28, 30, 36, 40])
def test_routed_launches_share_the_experts_in_use(plan, n):
    """A routed batch of n instances: workgroups for every compute unit (a
    slice of down its share of them), and for any number of experts in use,
    which the kernel alone knows, every tile has one owner; no workgroup walks
    more than an even share and a crossing (five tiles per lane) would cost."""
    for kind, args, tiles, cus in (("gateup", (16, 2880, 2880, 64, 2, 16), 180, 256),
                                   ("linear", (16, 2880, 2880, 64, 4), 180, 256),
                                   ("linear", (16, 512, 6656, 128, 4), 32, 128),     # two slices
                                   ("gateup", (16, 512, 64, 64, 2, 16), 4, 256)):
        p = plan(kind, *args, n, 1)
        assert p["wgs"] == min(cus, -(-n * tiles // p["tw"])) and p["wpb"] == 0
        for nv in range(1, n + 1):
            most = _cover(plan.ranges("routed_range", p["wgs"], p["wgs"], nv, tiles, p["tw"]), nv * tiles, tiles)
            assert most <= -(-nv * tiles // p["wgs"]) + 5 * p["tw"]
