"""The rules that choose between two kernels, held against measured times: each
takes the kernel that was the faster, over the range and not at single shapes.
The rules are host code without HIP and are compiled here by themselves."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1711_10275_amd", "csrc")

WRAP = """
#include "routes.h"
extern "C" int pool_table(int K, long long n_pairs, long long n_out, int pieces, int pb) {
  return sscn::pool_takes_table(K, n_pairs, n_out, (n_out + 63) / 64, pieces, pb);
}
extern "C" int narrow(int elem_bytes, int K, int kdim, int ncols, long long n_pairs, long long n_out) {
  return sscn::narrow_is_faster(elem_bytes, K, kdim, ncols, n_pairs, n_out);
}
extern "C" int point(int elem_bytes, int kdim, int ncols) {
  return sscn::point_is_faster(elem_bytes, kdim % 8 == 0, kdim, ncols);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "wrap.cpp").write_text(WRAP)
    so = str(d / "wrap.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.pool_table.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    lib.narrow.argtypes = [ctypes.c_int] * 4 + [ctypes.c_int64] * 2
    return lib


def _pieces(channels, dtype):
    """(pieces, pb) of a row as launch_pool forms them, of aligned tensors."""
    v = 4 if dtype == "f32" else 8
    pieces, pb = (channels // v, 3) if channels % v == 0 else (channels, 6)
    while pb and 1 << (pb - 1) >= pieces:
        pb -= 1
    return pieces, pb


# filter, rows written, pairs, channels, dtype, us of the table kernel, us of the walk
POOL = [
    (2, 25821, 100000, 64, "f32", 9.8, 38.2),  # average
    (2, 100000, 100000, 64, "f32", 12.7, 18.2),  # its gradient
    (3, 11547, 100000, 64, "f32", 14.5, 59.6),  # average
    (3, 100000, 100000, 16, "f32", 10.6, 18.6),  # its gradient
    (3, 100000, 100000, 36, "f32", 24.1, 19.1),  # its gradient
    (3, 32426, 275876, 32, "bf16", 10.5, 43.9),  # average
    (3, 20000, 20000, 13, "bf16", 13.7, 14.3),  # its gradient
    (4, 71432, 1000000, 64, "f32", 72.1, 303.1),  # average
    (4, 1000000, 1000000, 64, "f32", 296.7, 264.1),  # its gradient
    (4, 1000000, 1000000, 5, "f32", 135.9, 252.5),  # its gradient
    (3, 500000, 500000, 13, "f32", 59.7, 86.3),  # its gradient
    (4, 2000, 2000, 13, "f32", 23.8, 18.9),  # its gradient
    (4, 100000, 792014, 32, "f32", 30.7, 96.8),  # its gradient
    (5, 100000, 100000, 64, "f32", 98.2, 59.1),  # its gradient
    (5, 20000, 20000, 100, "f32", 43.0, 33.9),  # its gradient
    (6, 100000, 100000, 16, "f32", 118.6, 79.4),  # its gradient
    (6, 100000, 100000, 64, "f32", 340.3, 96.5),  # its gradient
    (6, 1000000, 1000000, 1, "f32", 893.7, 662.0),  # its gradient
    (8, 100000, 100000, 64, "f32", 1527.9, 195.7),  # its gradient
    (8, 100000, 100000, 100, "bf16", 7926.7, 360.3),  # its gradient
    (8, 1642, 100000, 64, "f32", 177.1, 646.5),  # average
    (2, 620, 2000, 100, "bf16", 19.8, 17.0),  # average
    (2, 2000, 2000, 100, "bf16", 15.6, 10.2),  # its gradient
    (3, 310, 2000, 100, "bf16", 54.7, 34.7),  # maximum
    (3, 9511, 67396, 33, "f32", 41.2, 34.6),  # average
    (3, 62481, 500000, 33, "f32", 61.1, 129.2),  # average
    (2, 100000, 100000, 33, "bf16", 21.1, 13.7),  # its gradient
    (8, 52, 2000, 13, "bf16", 201.9, 169.1),  # average
    (2, 136670, 500000, 20, "bf16", 30.3, 54.9),  # average
    (2, 274166, 1000000, 13, "bf16", 31.5, 104.8),  # maximum
]


def test_pool_rule_takes_the_faster_kernel(rules):
    for f, n_out, n_pairs, c, dtype, table, walk in POOL:
        got = bool(rules.pool_table(f ** 3, n_pairs, n_out, *_pieces(c, dtype)))
        assert got == (table < walk), (f, n_out, n_pairs, c, dtype)


def test_pool_rule_in_other_dimensions(rules):
    """Offsets, pairs and rows of 2- and 4-d fields."""
    for K, n_out, n_pairs, c, dtype, table, walk in [(4, 100000, 100000, 33, "bf16", 15.6, 12.5), (9, 100000, 223000, 33, "bf16", 28.3, 22.1),
                                                     (256, 79000, 400000, 8, "bf16", 229.7, 173.3)]:
        assert bool(rules.pool_table(K, n_pairs, n_out, *_pieces(c, dtype))) == (table < walk), (K, n_out, c)


def test_pool_rule_at_its_ends(rules):
    assert not rules.pool_table(8, 0, 100, *_pieces(64, "f32"))  # no pairs: nothing to look up
    assert not rules.pool_table(8, 0, 0, *_pieces(1, "f32"))
    assert rules.pool_table(1, 100, 100, *_pieces(1, "bf16"))


# reduction channels, columns, dtype, us of the per-site kernel, us of the general kernels
# (500k sites, or 1.96M where that is the closer pair)
POINT = [
    (36, 28, "f32", 34.2, 54.4), (36, 8, "f32", 22.3, 31.5), (20, 32, "f32", 25.1, 55.4), (12, 48, "f32", 26.6, 92.7),
    (8, 128, "f32", 67.0, 107.1), (24, 40, "f32", 75.2, 54.8), (13, 70, "f32", 61.2, 174.3), (70, 13, "f32", 68.2, 91.8),
    (33, 31, "f32", 60.1, 100.7), (5, 160, "f32", 95.7, 290.9), (70, 4, "f32", 145.7, 83.9), (70, 12, "f32", 63.3, 93.1), (33, 8, "f32", 174.8, 163.3),
    (44, 4, "f32", 133.9, 102.1), (44, 20, "f32", 144.8, 178.8), (50, 4, "f32", 401.8, 198.1), (50, 20, "f32", 362.9, 409.4),
    (60, 16, "f32", 178.0, 132.1), (100, 10, "f32", 270.7, 194.8), (100, 7, "f32", 243.1, 184.9),
    (40, 20, "bf16", 25.2, 30.8), (32, 20, "bf16", 23.3, 32.7), (16, 16, "bf16", 14.1, 25.2), (64, 12, "bf16", 24.9, 27.0),
    (80, 4, "bf16", 29.1, 28.1), (128, 6, "bf16", 34.2, 29.6), (200, 4, "bf16", 64.4, 46.6), (400, 2, "bf16", 118.0, 104.3),
    (32, 25, "bf16", 32.4, 30.2), (50, 20, "bf16", 35.4, 118.1), (70, 12, "bf16", 51.8, 78.2), (70, 4, "bf16", 145.4, 71.3),
    (100, 4, "bf16", 166.2, 95.4), (3, 64, "bf16", 28.2, 102.1),
]


def test_per_site_rule_takes_the_faster_kernel(rules):
    for kdim, ncols, dtype, here, general in POINT:
        assert bool(rules.point(4 if dtype == "f32" else 2, kdim, ncols)) == (here < general), (kdim, ncols, dtype)
    # fp32 rows taken as bf16 parts keep their rounding
    assert not any(rules.point(4, kdim, 4) for kdim in (16, 24, 32, 40, 64, 128))
    assert not rules.point(4, 65536, 65536)  # the product of the largest widths stays in range


# offsets, pairs, rows written, reduction channels, columns, dtype, us of the narrow kernel, us of the general kernels
NARROW = [
    (27, 1140000, 100000, 3, 32, "f32", 27.9, 204.6), (27, 1140000, 100000, 4, 96, "f32", 143.7, 285.4),
    (27, 220000, 20000, 7, 48, "f32", 48.0, 188.7), (27, 19000, 1799, 3, 32, "bf16", 24.7, 157.5),
    (27, 5700000, 500000, 7, 48, "bf16", 1143.8, 694.1), (27, 110303, 100000, 6, 64, "bf16", 102.3, 64.5),
    (27, 22080, 20000, 6, 32, "bf16", 23.0, 56.8), (27, 604300, 500000, 3, 128, "bf16", 468.6, 346.9),
    (27, 1959, 1799, 4, 96, "f32", 37.5, 25.3), (125, 1500000, 50000, 4, 8, "f32", 69.5, 177.7),
    (8, 20000, 6140, 6, 96, "bf16", 38.2, 73.6), (8, 20000, 6140, 1, 512, "bf16", 59.0, 41.2),
    (8, 20000, 6140, 4, 192, "f32", 36.5, 32.1), (8, 100000, 25821, 4, 192, "f32", 43.7, 67.2),
    (8, 500000, 136670, 5, 160, "f32", 129.2, 280.6), (8, 100000, 100000, 7, 128, "bf16", 73.5, 46.0),
    (8, 100000, 100000, 5, 96, "f32", 35.5, 63.5), (8, 1799, 1799, 1, 256, "bf16", 25.8, 21.7),
    (8, 500000, 500000, 7, 48, "bf16", 139.4, 123.3), (8, 1799, 1799, 4, 256, "f32", 36.3, 22.6), (8, 500000, 500000, 7, 96, "bf16", 186.1, 182.9),
    (8, 500000, 500000, 7, 96, "f32", 153.5, 206.6), (81, 2307196, 500000, 4, 16, "f32", 314.5, 158.3),
    (81, 457088, 100000, 4, 16, "f32", 79.1, 104.0), (81, 2307196, 500000, 1, 16, "f32", 118.8, 245.7),
    (81, 2307196, 500000, 5, 12, "bf16", 394.7, 228.7),
]


def test_narrow_rule_takes_the_faster_kernel(rules):
    for K, n_pairs, n_out, kdim, ncols, dtype, here, general in NARROW:
        got = bool(rules.narrow(4 if dtype == "f32" else 2, K, kdim, ncols, n_pairs, n_out))
        assert got == (here < general), (K, n_out, kdim, ncols, dtype)


def test_narrow_rule_keeps_within_the_lds(rules):
    """No more than 48 KB of weights and table, whatever the pairs."""
    for K in (1, 8, 27, 125, 512):
        for kdim in range(1, 8):
            for ncols in (1, 4, 5, 64, 300, 3000, 65536):
                if rules.narrow(4, K, kdim, ncols, K * 10 ** 6, 10 ** 6):
                    assert 4 * K * kdim * -(-ncols // 4) * 4 + 256 * K <= 48 * 1024
    assert not rules.narrow(4, 27, 8, 4, 10 ** 7, 10 ** 6) and not rules.narrow(4, 27, 7, 65536, 10 ** 7, 10 ** 6)
