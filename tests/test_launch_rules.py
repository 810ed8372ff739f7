"""The host's choices of sizes and kernel variants (csrc/rules.hpp), compiled for
the host and checked over the whole range of inputs, without a device."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1908_05944_amd", "csrc")
N_MAX = (1 << 26) - 1  # most balls of a call
INT_MAX = (1 << 31) - 1
RADII = [1, 1700, 1900, 1901, 2000, 2001, 2350, 2351, 2600, 2601, 3200, 3400, 3401, 5000, 8191]  # s_g, mA

WRAPPERS = """
#include "rules.hpp"
extern "C" {
int neighbour_slot(long long sgc, long long n) { return acx::neighbour_slot(sgc, n); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", f"-I{CSRC}", "-o", str(so),
                    str(src)], check=True)
    return ctypes.CDLL(str(so))


def _L(*a):
    return [ctypes.c_longlong(x) for x in a]


@pytest.mark.parametrize("n", [1, 300, 1 << 18, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 25) + 77, N_MAX])
def test_neighbour_rows_have_int32_indices(rules, n):
    for sgc in RADII:
        slot = rules.neighbour_slot(*_L(sgc, n))
        assert slot in (16, 32, 128)
        assert n * slot <= INT_MAX, (sgc, slot)  # the end of the last ball's row


def test_slots_where_they_fit(rules):
    for n in (1, 100000, (1 << 24) - 1):
        assert [rules.neighbour_slot(*_L(s, n)) for s in (1900, 1901, 2600, 2601, 3400, 3401)] == [16, 32, 32, 128, 128, 16]
