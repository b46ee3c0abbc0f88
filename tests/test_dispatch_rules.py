"""The size rules that choose between kernels, against the times of both sides.

rules.h is plain host code: it is compiled here by the host compiler.  Every
row of a table holds the measured microseconds of each choice at one shape;
the rule may not take one that is more than a few per cent slower than the
best (the spread between boxes is about 2%)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_35139_amd", "csrc")
SHIM = """
#include "rules.h"
extern "C" {
int expand_on_256(long M, long N, int K) { return cr::expand_on_256(M, N, K); }
int attention_queries(long N, int n_heads, int d_head, int fp32, long max_keys) {
  return cr::attention_queries(N, n_heads, d_head, fp32, max_keys);
}
int prefetch(long wgs, int queries, long range, long total) {
  return cr::prefetch_pays(range, total) && cr::prefetch_fits(wgs, queries);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


# rows, columns, K: us on 128-column tiles, on 256-column tiles
EXPAND = [
    (200, 18432, 512, 13.8, 20.9), (1100, 18432, 512, 41.7, 44.1), (1500, 18432, 512, 50.5, 47.2),
    (1920, 18432, 512, 63.4, 70.1), (2690, 18432, 512, 86.0, 94.3), (3200, 18432, 512, 101.3, 97.0),
    (3600, 18432, 512, 110.3, 116.5), (4000, 18432, 512, 133.7, 124.7),
    (7300, 18432, 512, 219.9, 223.4), (8192, 18432, 512, 263.0, 253.0),
    (512, 18432, 1024, 43.2, 34.1), (800, 18432, 1024, 46.4, 66.9), (1280, 18432, 1024, 69.1, 73.8),
    (2300, 18432, 1024, 121.3, 111.6), (4096, 18432, 1024, 201.3, 189.3),
    (5120, 18432, 1024, 242.8, 224.9), (8192, 18432, 1024, 398.7, 349.8),
    (57, 65536, 1024, 28.0, 36.2), (128, 65536, 1024, 33.0, 40.1), (135, 65536, 1024, 47.8, 40.5),
    (320, 65536, 1024, 70.5, 75.1), (640, 65536, 1024, 117.4, 112.7),
    (5120, 65536, 1024, 880.5, 762.3),
    (1920, 18432, 256, 46.3, 54.4), (3200, 18432, 256, 74.3, 75.9), (8192, 18432, 128, 140.8, 176.3),
    (200, 15360, 512, 9.8, 20.1), (2000, 15360, 1024, 89.9, 78.8),
    (1500, 18432, 1536, 113.4, 96.0), (2690, 18432, 2048, 247.6, 229.7),
    (800, 18432, 2048, 77.0, 107.5),
]


@pytest.mark.parametrize("M,N,K,small,wide", EXPAND)
def test_output_add_takes_the_faster_tiles(rules, M, N, K, small, wide):
    taken = wide if rules.expand_on_256(ctypes.c_long(M), ctypes.c_long(N), K) else small
    assert taken <= 1.05 * min(small, wide)


MB = 1 << 20
# attention workgroups, their queries, bytes to prefetch, bytes of the repairer:
# us of the call without, with
PREFETCH = [
    (32, 32, 26 * MB, 267 * MB, 384.6, 347.2), (144, 32, 26 * MB, 267 * MB, 481.6, 488.1),
    (128, 32, 26 * MB, 267 * MB, 444.8, 419.8), (192, 32, 26 * MB, 267 * MB, 510.5, 494.3),
    (208, 32, 26 * MB, 267 * MB, 520.0, 527.0), (224, 64, 26 * MB, 267 * MB, 704.9, 676.5),
    (384, 64, 26 * MB, 267 * MB, 962.0, 898.3), (480, 64, 26 * MB, 267 * MB, 1180.2, 1137.0),
    (208, 128, 26 * MB, 267 * MB, 1022.3, 980.7), (576, 128, 26 * MB, 267 * MB, 2215.9, 2175.7),
    # a repairer that stays in the cache
    (64, 32, 26 * MB, 162 * MB, 176.1, 181.2), (96, 32, 14 * MB, 82 * MB, 131.0, 134.3),
    # ranges that take longer to read than the attention
    (64, 32, 100 * MB, 512 * MB, 321.7, 328.2), (64, 32, 164 * MB, 604 * MB, 333.4, 355.6),
    (64, 32, 292 * MB, 989 * MB, 473.5, 579.7), (320, 128, 292 * MB, 989 * MB, 1671.5, 1800.2),
    (16, 32, 6 * MB, 53 * MB, 149.0, 152.0),
    # many rounds
    (1888, 128, 26 * MB, 267 * MB, 8301.8, 8369.6),
]


@pytest.mark.parametrize("wgs,q,range_,total,without,with_", PREFETCH)
def test_weights_are_prefetched_where_that_is_faster(rules, wgs, q, range_, total, without, with_):
    on = rules.prefetch(ctypes.c_long(wgs), q, ctypes.c_long(range_), ctypes.c_long(total))
    assert (with_ if on else without) <= 1.015 * min(without, with_)


# tokens, heads, d_head, fp32, keys of the longest row: us on 32-, 64- and 128-query tiles
ATTENTION = [
    (200, 16, 64, 0, 200, 5.5, 6.1, None),
    (1024, 16, 64, 0, 1024, None, 9.4, 12.5), (1024, 16, 64, 0, 100, None, 7.5, 10.0),
    (1500, 16, 64, 0, 1500, None, 15.8, 17.4), (2000, 16, 64, 0, 200, None, 13.9, 12.0),
    (2500, 8, 64, 0, 2500, None, 17.6, 24.7), (2500, 8, 64, 0, 800, None, 16.5, 24.4),
    (2500, 8, 64, 0, 512, None, 12.6, 9.4), (2500, 8, 64, 0, 256, None, 10.5, 7.0),
    (2500, 8, 64, 0, 100, None, 11.4, 10.4), (3600, 8, 64, 0, 100, None, 12.9, 11.0),
    (4000, 8, 64, 0, 300, None, 18.1, 15.2), (4000, 8, 64, 0, 4000, None, 32.3, 37.1),
    (1500, 16, 32, 0, 1500, None, 10.2, 12.9), (1500, 16, 32, 0, 400, None, 13.0, 13.8),
    (3000, 16, 32, 0, 3000, None, 26.6, 23.3),
    (2048, 8, 64, 1, 2048, 54.1, None, 130.4), (3900, 8, 64, 1, 100, 30.5, None, 34.6),
    (4096, 16, 64, 1, 4096, 359.5, None, 302.4), (2560, 16, 64, 1, 2560, 156.0, None, 168.5),
]


@pytest.mark.parametrize("N,heads,dh,fp32,keys,t32,t64,t128", ATTENTION)
def test_attention_takes_the_faster_query_tiles(rules, N, heads, dh, fp32, keys, t32, t64, t128):
    q = rules.attention_queries(ctypes.c_long(N), heads, dh, fp32, ctypes.c_long(keys))
    times = {32: t32, 64: t64, 128: t128}
    assert times[q] is not None and times[q] <= 1.02 * min(t for t in times.values() if t)
