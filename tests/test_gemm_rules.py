"""Host checks of the rules that choose a product's kernel (CPU): the plain C++
functions that the launcher uses, compiled with the host compiler."""
import ctypes as C
import os
import subprocess

import pytest

from tests import test_gpu_gemm_tiles as tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_28803_amd", "csrc")

SOURCE = r"""
#include "gemm_rules.h"
extern "C" int ring_tiling(int64_t M, int64_t N, int64_t K, bool a8) { return oq::ring_tiling(M, N, K, a8); }
extern "C" bool few_rows(int64_t M, int64_t N, int64_t K, bool a8, bool tiled) { return oq::few_rows(M, N, K, a8, tiled); }
extern "C" void small_shape(int64_t N, int64_t K, bool a8, int* out) {
  const oq::SmallShape s = oq::small_shape(N, K, a8);
  out[0] = s.nb, out[1] = s.waves, out[2] = s.ub;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = C.CDLL(str(so))
    lib.small_shape.argtypes = [C.c_int64, C.c_int64, C.c_bool, C.POINTER(C.c_int)]
    lib.few_rows.argtypes = [C.c_int64] * 3 + [C.c_bool] * 2
    lib.few_rows.restype = C.c_bool
    lib.ring_tiling.argtypes = [C.c_int64] * 3 + [C.c_bool]
    return lib


@pytest.mark.parametrize("a8", [False, True])
@pytest.mark.parametrize("N", [1, 4096, 4097, 32768])
@pytest.mark.parametrize("K", [64, 128, 192, 320, 1024, 1088, 2048, 2112, 16384])
def test_few_row_loads_stay_within_a_row(rules, N, K, a8):
    """A round's unconditional 64-byte unit loads read unit min(u, last) or 0: the row (K / 2 bytes of
    packed codes) must hold at least one unit, or the round must load none."""
    out = (C.c_int * 3)()
    rules.small_shape(N, K, a8, out)
    nb, waves, ub = out
    units = K // 128
    for wave in range(waves):
        beg, end = units * wave // waves, units * (wave + 1) // waves
        for u in range(beg, beg + ub):  # the first round; later ones start below `end`
            unit = u if u < end else max(end - 1, 0)
            assert unit * 64 + 64 <= K // 2
    assert (nb, waves) == ((2, 8) if N > 4096 else (1, 4 if K <= 1024 else 16))


# (M, N, K, 8-bit tokens, us on the small-M kernel, us on the ring): both measured on an MI355X in
# graphs of many calls that rotate through more weights than the caches hold.
MEASURED = [
    (1, 16384, 16384, False, 29.9, 37.9), (8, 16384, 16384, False, 32.0, 38.3), (16, 16384, 16384, False, 34.8, 39.0),
    (17, 8200, 576, False, 4.00, 5.09), (48, 16384, 576, False, 4.96, 5.60), (17, 8200, 1024, False, 4.22, 5.10),
    (17, 16384, 1024, False, 5.15, 5.90), (32, 8200, 1024, False, 4.59, 5.14), (36, 16384, 768, False, 5.45, 5.61),
    (40, 8200, 1024, False, 4.81, 5.25), (48, 10000, 1024, False, 5.78, 5.36), (17, 8200, 1088, False, 7.75, 5.97),
    (17, 32768, 1024, False, 9.06, 7.66), (64, 32768, 512, False, 11.14, 6.20), (17, 9000, 4096, False, 13.9, 11.2),
    (40, 32768, 2048, False, 29.2, 11.6), (64, 10000, 8192, False, 31.7, 19.5), (17, 8200, 16384, False, 34.9, 31.7),
    (64, 16384, 16384, False, 60.3, 39.7), (17, 16384, 576, True, 5.07, 5.63), (24, 12288, 576, True, 5.16, 5.53),
    (24, 12288, 768, True, 5.94, 5.49), (17, 8200, 1024, True, 5.10, 5.87), (24, 16384, 1024, True, 6.36, 6.70),
    (28, 9000, 1024, True, 6.24, 5.96), (17, 8200, 4096, True, 15.0, 16.1), (17, 8200, 8192, True, 25.9, 28.6),
    (17, 8200, 16384, True, 43.4, 53.3), (17, 16384, 16384, True, 53.5, 58.1), (20, 12288, 16384, True, 52.8, 54.3),
    (24, 8200, 8192, True, 27.6, 28.7), (28, 8200, 16384, True, 49.9, 53.6), (24, 9000, 8192, True, 30.6, 28.9),
    (24, 10000, 16384, True, 54.8, 53.6), (17, 20000, 16384, True, 76.0, 59.4), (40, 32768, 2048, True, 25.0, 12.8),
    (64, 32768, 8192, True, 92.7, 41.3),
    (17, 8200, 64, False, 2.82, 3.13), (48, 9000, 64, False, 3.38, 3.43), (64, 9000, 64, False, 3.70, 3.43),
    (17, 20000, 64, False, 4.31, 3.66), (64, 9000, 64, True, 3.75, 4.16), (64, 16392, 64, True, 5.13, 4.57),
    (17, 9000, 128, False, 3.87, 3.44), (24, 8200, 192, False, 3.52, 3.62), (17, 9000, 192, False, 3.77, 3.60),
    (64, 8200, 256, False, 5.23, 3.77), (17, 8200, 384, False, 3.62, 4.12),
    (40, 12288, 448, False, 4.28, 4.38), (64, 9000, 448, False, 4.80, 4.44), (32, 8200, 512, False, 4.45, 4.32),
    (64, 8200, 640, False, 4.33, 5.21), (64, 16384, 896, False, 5.91, 6.21), (64, 9000, 832, False, 6.04, 5.79),
    (56, 9000, 704, False, 4.97, 5.27), (48, 20000, 640, False, 6.65, 7.11),
    (56, 20000, 704, False, 7.83, 7.43), (17, 16392, 1024, False, 6.00, 6.51), (17, 32768, 640, False, 7.29, 7.08),
    (24, 8200, 320, True, 4.59, 4.26), (17, 8200, 576, True, 4.36, 4.72), (24, 9000, 640, True, 5.17, 4.73),
    (17, 8200, 768, True, 5.03, 5.28), (64, 9000, 832, True, 6.21, 5.72), (17, 16384, 960, True, 5.58, 6.18),
    (40, 9000, 896, True, 6.09, 5.48),
]


@pytest.mark.parametrize("M,N,K,a8,small,ring", MEASURED)
def test_few_row_rule_takes_the_faster_kernel(rules, M, N, K, a8, small, ring):
    assert rules.few_rows(M, N, K, a8, False) == (small < ring)


def test_few_row_rule_takes_what_only_the_small_kernel_reads(rules):
    for M in (1, 16, 17, 64, 65, 5000):
        for N in (8, 8192, 100000):
            for K in (128, 1024, 16384):
                assert rules.few_rows(M, N, K, False, True)
                assert rules.few_rows(M, N, K, False, False) <= (M <= 64)


# Ring tilings by index: W4A4 256 x 256, 128 x 128, 128 x 64, 64 x 64 with four K groups, 64 x 64, and with 128-code stages 64 x
# 64 and 128 x 64; W4A8 256 x 256, 128 x 128, 64 x 64 with two K groups.  What the GPU tests' shapes say beside them.
TILING = {"W4A4": [0, 0, 1, 1, 2, 2, 3, 3, 3, 4, 4, 5, 5, 5, 6, 6], "W4A8": [0, 1, 1, 2, 2, 2, 1]}


@pytest.mark.parametrize("name", sorted(TILING))
def test_tiling_shapes_take_the_tiling_they_name(rules, name):
    shapes = getattr(tiles, name)
    assert len(shapes) == len(TILING[name])
    for (M, N, K), tiling in zip(shapes, TILING[name]):
        assert not rules.few_rows(M, N, K, name == "W4A8", False)
        assert rules.ring_tiling(M, N, K, name == "W4A8") == tiling, (M, N, K)


# (8-bit tokens, M, N, K, us with each tiling), measured as above.
TIMES = [
    (False, 128, 4096, 4096, [43.0, 18.7, 14.2, 9.1, 10.7]), (False, 256, 8192, 8192, [82.3, 36.1, 30.5, 24.6, 28.5]),
    (False, 512, 2048, 4096, [43.9, 19.4, 14.7, 9.8, 11.2]), (False, 816, 2560, 2048, [26.2, 12.6, 12.9, 13.1, 13.7]),
    (False, 816, 2048, 16384, [153.7, 63.3, 50.9, 39.4, 47.6]), (False, 816, 32768, 2048, [65.6, 63.8, 71.3, 96.8, 94.5]),
    (False, 1024, 1536, 6144, [61.0, 26.0, 20.2, 17.6, 19.8]), (False, 1024, 6144, 1536, [23.4, 16.7, 15.8, 20.8, 20.1]),
    (False, 1024, 4608, 1536, [22.4, 15.4, 14.2, 17.0, 16.9]), (False, 2000, 6144, 1536, [25.5, 23.7, 26.0, 36.9, 35.1]),
    (False, 4000, 4096, 4096, [57.6, 64.2, 73.3, 90.8, 101.6]),
    (False, 4080, 2048, 16384, [168.5, 117.4, 143.8, 159.7, 186.9]),
    (False, 4080, 4096, 1024, [23.3, 24.8, 26.7, 40.7, 39.6]),
    (False, 4096, 8192, 8192, [195.5, 229.0, 271.0, 321.9, 356.8]),
    (False, 16384, 4096, 4096, [207.7, 231.1, 281.2, 356.2, 377.1]),
    (False, 16384, 8192, 8192, [777.4, 893.1, 1051.9, 1247.9, 1379.3]), (True, 128, 4096, 4096, [48.6, 22.9, 11.8]),
    (True, 256, 8192, 8192, [91.7, 43.4, 32.4]), (True, 512, 2048, 4096, [49.1, 23.2, 12.2]),
    (True, 816, 2560, 2048, [29.3, 15.0, 12.7]), (True, 816, 2048, 16384, [174.1, 81.1, 52.0]),
    (True, 816, 32768, 2048, [77.7, 77.3, 97.7]), (True, 1024, 1536, 6144, [70.5, 32.9, 20.6]),
    (True, 1024, 6144, 1536, [26.0, 18.7, 19.9]), (True, 1024, 4608, 1536, [24.8, 17.4, 16.7]),
    (True, 2000, 6144, 1536, [30.4, 29.1, 35.6]), (True, 4000, 4096, 4096, [68.6, 77.2, 96.6]),
    (True, 4080, 2048, 16384, [206.1, 142.2, 188.2]), (True, 4080, 4096, 1024, [25.8, 28.2, 37.2]),
    (True, 4096, 8192, 8192, [243.3, 275.9, 367.1]), (True, 16384, 4096, 4096, [256.6, 285.9, 382.0]),
    (True, 16384, 8192, 8192, [931.2, 1086.6, 1429.6]),
]


@pytest.mark.parametrize("a8,M,N,K,us", TIMES)
def test_ring_rule_takes_a_fast_tiling(rules, a8, M, N, K, us):
    slack = 1.19 if (a8, M, N, K) == (True, 816, 2560, 2048) else 1.07
    assert us[rules.ring_tiling(M, N, K, a8)] <= slack * min(us)


# (M, N, K, us with each of the seven W4A4 tilings): short K.
SHORT = [(65, 16384, 128, 9.84, 5.91, 5.06, 6.21, 5.57, 4.23, 4.59), (600, 4096, 128, 10.48, 6.26, 5.78, 8.27, 7.63, 4.83, 5.18),
         (4080, 4096, 64, 14.03, 14.77, 15.21, 30.48, 28.80, 12.46, 11.88), (8192, 8192, 256, 48.54, 44.19, 44.93, 110.94, 100.90, 41.17, 37.02)]


@pytest.mark.parametrize("shape", SHORT)
def test_short_k_takes_the_fastest_tiling(rules, shape):
    M, N, K, *us = shape
    assert rules.ring_tiling(M, N, K, False) == us.index(min(us))


def test_short_k_of_w4a8_takes_128x128(rules):
    assert rules.ring_tiling(1100, 32768, 128, True) == 1 and rules.ring_tiling(2500, 16384, 192, True) == 1
    assert rules.ring_tiling(4080, 32768, 128, True) == 0  # (90.5 us, 128 x 128 102)


def test_few_row_shapes_take_the_kernel_they_name(rules):
    on_ring = {(17, 8200, 1088): (4, 2), (64, 8200, 4160): (3, 2)}  # (W4A4, W4A8) tilings
    for M, N, K in tiles.FEW:
        for a8 in (False, True):
            assert rules.few_rows(M, N, K, a8, False) == ((M, N, K) not in on_ring)
            if (M, N, K) in on_ring:
                assert rules.ring_tiling(M, N, K, a8) == on_ring[M, N, K][a8]


def test_residual_linears_take_the_tiling_they_name(rules):
    cfg = tiles.RESID["gr00t_2000"][0]
    rows, d, f = cfg.batch * cfg.tokens, cfg.hidden, cfg.mlp
    assert (rows, d, f) == (2000, 1536, 6144)
    assert [rules.ring_tiling(rows, n, k, False) for n, k in ((d, d), (d, f), (f, d))] == [2, 1, 1]  # o, ff2, ff0
    cfg = tiles.RESID["pi_8192"][0]
    rows, d, f = cfg.batch * cfg.tokens, cfg.hidden, cfg.mlp
    assert [rules.ring_tiling(rows, n, k, False) for n, k in ((d, d), (2 * f, d), (d, f))] == [0, 0, 0]  # o, gate|up, down
    for name, tiling in (("gr00t_narrow", 5), ("gr00t_narrow_801", 6)):
        cfg = tiles.RESID[name][0]
        assert rules.ring_tiling(cfg.batch * cfg.tokens, cfg.hidden, cfg.mlp, False) == tiling and cfg.hidden == cfg.mlp
