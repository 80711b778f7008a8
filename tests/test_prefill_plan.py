"""The split of a prefill chunk (csrc/prefill_plan.h, host C++ over sizes and
compute units), compiled here with g++ and checked without a GPU."""
import shutil

import pytest

from qmlp_testutil import PREFILL_PLAN_SRC, host_library

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return host_library(PREFILL_PLAN_SRC, tmp_path_factory.mktemp("plan"))


@pytest.mark.parametrize("cus", [32, 64, 128, 256])
def test_tiles_and_slices_divide_the_chunk(plan, cus):
    for M in range(128, 2049, 128):
        for d in (128, 2560, 4096, 6144):
            for f in (64, 320, 768, 2048, 8320, 9728, 12288, 16384):
                bm, hc = plan.tile_bm(M, f, cus), plan.tile_hc(M, f, cus)
                assert (bm, hc) in ((256, 128), (256, 64), (128, 64)) and M % bm == 0 and f % hc == 0
                S, most = plan.slices(M, d, f, cus), plan.slices_most(M, d, f)
                assert 1 <= S <= most <= 8 and f % (64 * S) == 0   # whole 64-wide steps per slice
                bm = 256 if M % 256 == 0 else 128
                assert S == 1 or (M // bm) * (d // 128) * S <= (cus if bm == 256 else 2.5 * cus)


def test_rules_count_the_compute_units_of_the_device(plan):
    """The rounds over the chip decide, so a partition of it chooses otherwise:
    a 256-token chunk of the 4B shape, and slices that fill the compute units
    there are."""
    assert (plan.tile_bm(256, 9728, 256), plan.tile_hc(256, 9728, 256)) == (256, 64)
    assert (plan.tile_bm(256, 9728, 128), plan.tile_hc(256, 9728, 128)) == (256, 128)
    assert [plan.slices(512, 2560, 9728, cus) for cus in (32, 64, 128, 256)] == [1, 1, 2, 4]
