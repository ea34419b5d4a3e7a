"""Host checks of the products' index arithmetic (CPU): the plain C++ rules that
the kernels and launchers use, compiled with the host compiler."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_28803_amd", "csrc")

SOURCE = r"""
#include "gemm_rules.h"
extern "C" int begin(int nu, int wave, int waves) { return oq::small_begin(nu, wave, waves); }
extern "C" int unit(int u, int uend) { return oq::small_unit(u, uend); }
extern "C" int piece(int nu, int quarter) { return oq::small_piece(nu, quarter); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 1024, 1088, 2048, 2112, 16320, 16384])
@pytest.mark.parametrize("waves,ub", [(4, 2), (8, 1), (8, 2), (8, 4), (16, 1), (16, 2)])
def test_few_row_loads_stay_within_a_row(rules, K, waves, ub):
    """Every 16-byte load of the few-row product lies inside the row it reads (K / 2 bytes of
    packed codes, K bytes of 8-bit codes), also where a row holds less than one unit, and the
    waves' units cover K exactly once."""
    nu = K // 128
    seen = []
    for wave in range(waves):
        beg, end = rules.begin(nu, wave, waves), rules.begin(nu, wave + 1, waves)
        seen += range(beg, end)
        for u0 in range(beg, max(end, beg + 1), ub):
            for u in range(u0, u0 + ub):
                uu = rules.unit(u, end)
                assert u >= end or uu == u
                for quarter in range(4):
                    p = rules.piece(nu, quarter)
                    assert nu == 0 or p == 16 * quarter
                    assert 0 <= uu * 64 + p and uu * 64 + p + 16 <= K // 2
                    for c in range(2):
                        assert uu * 128 + 2 * p + 16 * c + 16 <= K
    assert seen == list(range(nu))
