"""The pair counts of two-level binning (csrc/pair_count.h), compiled for the
host: packed sums that pass 2^32 pairs, in any grouping, keep and drop the
entries that sums of Python integers keep and drop, and no coarse pair is
placed past the capacity."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2605_06876_amd", "csrc")
PROGRAM = """
#define __host__
#define __device__
#define __forceinline__ inline
#include "pair_count.h"
// groups of `group` entries summed first, then every entry placed after the groups before its own
extern "C" void place(int64_t n, const uint64_t *c, uint64_t cap, int64_t group, uint8_t *kept, uint8_t *crosses,
                      uint64_t *at_out, uint64_t *all) {
    uint64_t pre = 0;
    for (int64_t g = 0; g < n; g += group) {
        const int64_t end = g + group < n ? g + group : n;
        uint64_t sum = 0;
        for (int64_t i = g; i < end; i++) {
            const uint64_t at = sat_add(pre, sum);
            const PairCut cut = pair_cut(at, c[i], cap);
            kept[i] = cut.kept;
            crosses[i] = cut.crosses;
            at_out[i] = at;
            sum = sat_add(sum, c[i]);
        }
        pre = sat_add(pre, sum);
    }
    *all = pre;
}
"""


@pytest.fixture(scope="module")
def place(tmp_path_factory):
    d = tmp_path_factory.mktemp("pair_count")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "p.so"), str(d / "p.cpp")], check=True)
    fn = ctypes.CDLL(str(d / "p.so")).place

    def call(bins, coarse, cap, group):
        c = (bins.astype(np.uint64) << np.uint64(32)) | coarse.astype(np.uint64)
        n = len(c)
        kept, crosses = np.zeros(n, np.uint8), np.zeros(n, np.uint8)
        at, all_ = np.zeros(n, np.uint64), ctypes.c_uint64()
        ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        fn(ctypes.c_int64(n), ptr(c), ctypes.c_uint64(cap), ctypes.c_int64(group), ptr(kept), ptr(crosses), ptr(at),
           ctypes.byref(all_))
        return kept, crosses, at, all_.value
    return call


MAX_CAP = 0xFFFFFFFE


@pytest.mark.parametrize("group", [1, 64, 2048])
@pytest.mark.parametrize("cap", [1 << 22, 19_200_000, MAX_CAP])
@pytest.mark.parametrize("n,bins,coarse", [
    (600_000, 8160, 510),            # every entry over a 1920x1080 view: wraps once and is over the capacity again
    (1_200_000, 8160, 8160),
    (12_000, 1 << 22, 1 << 18),      # the largest view, coarse counts past 2^32 as well
    (12_000, 1 << 22, 1 << 22),
    (526_345, 8160, 8160),           # 2^32 + 7,904 bins: the sum just wraps
    (1000, 4_294_967, 1),            # 2^32 - 296: it just does not
])
def test_counts_past_32_bits(place, n, bins, coarse, cap, group):
    b, c = np.full(n, bins, np.int64), np.full(n, coarse, np.int64)
    b[::7] = c[::7] = 0              # culled entries
    b[1::11] //= 3
    c[1::11] = np.minimum(c[1::11], b[1::11])
    end = np.cumsum(b)               # (below 2^63)
    off, coff = end - b, np.cumsum(c) - c
    kept, crosses, at, all_ = place(b, c, cap, group)
    np.testing.assert_array_equal(kept, (b > 0) & (end <= cap))
    np.testing.assert_array_equal(crosses, (b > 0) & (off <= cap) & (end > cap))
    k = kept.astype(bool)
    np.testing.assert_array_equal(at[k] & np.uint64(0xFFFFFFFF), coff[k].astype(np.uint64))
    assert not k.any() or int((coff + c)[k].max()) <= cap
    assert all_ >> 32 == min(int(end[-1]), 0xFFFFFFFF)
    assert (all_ >> 32 <= cap) == (int(end[-1]) <= cap)
