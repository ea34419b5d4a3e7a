"""Host checks of the rules that choose a product's kernel (CPU): the plain C++
functions that the launcher uses, compiled with the host compiler."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_28803_amd", "csrc")

SOURCE = r"""
#include "gemm_rules.h"
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
