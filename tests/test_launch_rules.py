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
int neighbour_slot(long long sgc, long long n, int recorded) { return acx::neighbour_slot(sgc, n, recorded != 0); }
int tet_slab(long long sgc, int gshift, int groups, long long most) { return acx::tet_slab(sgc, gshift, groups, most); }
int counts_triangles_in(long long left, long long pairs, long long n, long long E, long long Nn, long long g, long long cap) {
    return acx::counts_triangles_in(left, pairs, n, E, Nn, g, cap);
}
int counts_triangles(long long pairs) { return acx::counts_triangles(pairs); }
int has_index(long long total) { return acx::has_index(total); }
int inc_passes(long long n) { return acx::inc_buckets(n).passes; }
int inc_shift(long long n) { return acx::inc_buckets(n).shift; }
int group_shift(long long n, int slot, long long edges) { return acx::group_shift(n, slot, edges); }
int kernel_radius(long long sgc, long long large, long long n) { return (int)acx::kernel_radius(sgc, large, n); }
int later_counted(int later) { return acx::later_counted(later); }
int long_rows(long long pairs, long long edges) { return acx::long_rows(pairs, edges); }
double full_cell(long long n, long long ncell, int side) { return acx::full_cell(n, ncell, side); }
int tet_split(int groups) { return acx::tet_split(groups); }
int tests_split(int groups) { return acx::tests_split(groups); }
int rows_split(int parts) { return acx::rows_split(parts); }
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
        for recorded in (0, 1):
            slot = rules.neighbour_slot(*_L(sgc, n), recorded)
            assert slot in (16, 32, 128)
            assert n * slot <= INT_MAX, (sgc, slot)  # the end of the last ball's row


def test_slots_where_they_fit(rules):
    for n in (1, 100000, (1 << 24) - 1):
        assert [rules.neighbour_slot(*_L(s, n), 0) for s in (1900, 1901, 2600, 2601, 3400, 3401)] == [16, 32, 32, 128, 128, 16]
        assert [rules.neighbour_slot(*_L(s, n), 1) for s in (1900, 1901, 2600, 2601, 3400, 3401)] == [16, 32, 32, 16, 16, 16]


def test_a_few_large_balls_do_not_choose_the_kernels(rules):
    for n in (32, 1024, 100000, 2000000, N_MAX):
        for sgc, part in ((1700, 0), (2350, 0), (2600, 0), (2601, 32), (3000, 32), (3001, 1024), (3400, 1024), (3401, 0), (8191, 0)):
            for large in (1, n // 1024, n // 1024 + 1, n // 32, n // 32 + 1):
                few = part > 0 and large <= n // part
                got = rules.kernel_radius(*_L(sgc, large, n))
                assert got == (2000 if few else sgc), (n, sgc, large)
                if few:
                    assert rules.neighbour_slot(*_L(got, n), 0) == rules.neighbour_slot(*_L(got, n), 1) == 32
    assert rules.kernel_radius(*_L(2750, 1, 31)) == 2750


@pytest.mark.parametrize("n", [1, 300, 1 << 18, 40000000, 43600000, 43700000, 1 << 25, 1 << 26])
def test_tetrahedron_slabs_have_int32_indices(rules, n):
    for gshift in range(9):
        groups = ((n - 1) >> gshift) + 1
        for sgc in RADII:
            for most in (0, 1000000):
                cap = rules.tet_slab(*_L(sgc), gshift, groups, *_L(most))
                # (loops over a group's tetrahedra step a block past its last)
                assert 1 <= cap and cap * groups + 256 <= INT_MAX, (gshift, sgc, cap)


def test_slab_sizes_where_they_fit(rules):
    want = {1900: 8, 2000: 8, 2001: 16, 2350: 16, 2351: 48, 2600: 48, 2601: 16, 5000: 16}
    for sgc, ball in want.items():
        for gshift, groups in ((4, 20), (8, 20000)):
            cap = (ball << gshift) + (64 if sgc <= 2000 else 320)
            for most in (0, cap, cap + 1):
                assert rules.tet_slab(*_L(sgc), gshift, groups, *_L(most)) == max(cap, most)


def test_pairs_past_their_room_are_counted(rules):
    assert not rules.counts_triangles(*_L(1 << 28)) and rules.counts_triangles(*_L((1 << 28) + 1))


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 511, 512, 513, 4001, 1 << 17, (1 << 17) + 1, 200000, 1 << 18,
                               (1 << 18) + 1, 400000, 3000000, (1 << 25) + 1, N_MAX])
def test_buckets_of_the_corner_sort(rules, n):
    """Every ball id fits in the sorted bits, a bucket's balls in its counters, and
    there are no more blocks than some hundreds or than whole buckets."""
    passes, shift = rules.inc_passes(*_L(n)), rules.inc_shift(*_L(n))
    assert 1 <= passes and 0 <= shift <= 9
    assert (n - 1) >> (shift + 8 * passes) == 0
    assert passes == 1 or (n - 1) >> (9 + 8 * (passes - 1)) > 0  # no pass too many
    assert ((n - 1) >> shift) + 1 <= max(256, (n + 511) // 512)


def test_groups(rules):
    """Ordinary builds keep their groups; long rows in few balls make them smaller."""
    for n, slot, row, want in ((300, 16, 4, 4), (100000, 16, 4, 6), (100000, 128, 21, 4), (3000000, 16, 4, 8),
                               (3000, 32, 10, 4), (300, 16, 60, 0), (3000, 16, 200, 0), (60000, 16, 200, 3),
                               (70000, 16, 200, 4), (N_MAX, 32, 30, 8)):
        got = rules.group_shift(*_L(n), slot, *_L(n * row))
        assert got == want, (n, slot, row, got)
    assert rules.group_shift(*_L(1), 16, *_L(0)) == 4


@pytest.mark.parametrize("parts", [1, 17, 128, 129, 4095, 4096, 4097, N_MAX])
def test_blocks_of_a_part(rules, parts):
    assert rules.rows_split(parts) == min(32, max(1, 4096 // parts))
    assert rules.tests_split(parts) == min(32, max(8, 4096 // parts))


def test_pairs_on_fixed_scratch(rules):
    def counted(left, pairs, n=1000, E=4000, Nn=8000, groups=63, cap=192):
        return bool(rules.counts_triangles_in(*_L(left, pairs, n, E, Nn, groups, cap)))

    rest = 40 * 1000 + 33 * 4000 + 4 * 8000 + (64 + 16 * 192) * 63 + (1 << 20)
    assert not counted(rest + 37 * 5000, 5000) and counted(rest + 37 * 5000 - 1, 5000)
    assert counted(rest - 1, 1) and counted(0, 100)  # nothing left: the triangles need the least
    assert counted(1 << 40, (1 << 28) + 1)


def test_totals_leave_room_for_a_block(rules):
    """The largest radix tile (2,048 items) and two blocks past an accepted total
    are still int32 indices."""
    assert not rules.has_index(*_L(INT_MAX)) and rules.has_index(*_L(INT_MAX - 4096))
    for total in range(INT_MAX - 5000, INT_MAX):
        assert not rules.has_index(*_L(total)) or total + 2048 + 512 <= INT_MAX


def test_long_rows(rules):
    """On both sides of 16 later entries a row, and at the largest totals."""
    for edges in (0, 1, 100, 35525, INT_MAX - 4096):
        assert not rules.long_rows(*_L(8 * edges, edges)) and rules.long_rows(*_L(8 * edges + 1, edges))


def test_later_entries_of_the_edges_held(rules):
    """Their sum is an int32 for rows of any length, and still says which are long."""
    for later in (0, 1, 64, 8192, 8193, (1 << 22) - 1, 1 << 22, 5000000, N_MAX):
        got = rules.later_counted(later)
        assert 512 * got <= INT_MAX and (got == later or later > got > 8192)


def test_slices_of_a_group(rules):
    for groups, want in ((1, 5), (128, 5), (129, 4), (1000, 2), (2048, 1), (2049, 0), (4097, 0), (N_MAX, 0)):
        assert rules.tet_split(groups) == want, groups
        for sgc in RADII:
            assert rules.tet_slab(*_L(sgc), 0, groups << want, *_L(0)) * (groups << want) <= INT_MAX


def test_full_cells(rules):
    """2.5 times the mean in a molecule's own box; the density where most cells are empty."""
    rules.full_cell.restype = ctypes.c_double
    assert rules.full_cell(*_L(3000000, 3800000), 1800) == pytest.approx(2.5 * 3 / 3.8)
    assert rules.full_cell(*_L(159284, 262144), 9000) == pytest.approx(0.06 * 729)
    for side in (1, 700, 1800, 9000, 60000, 1 << 20):
        assert rules.full_cell(*_L(1, 1 << 30), side) > 0
