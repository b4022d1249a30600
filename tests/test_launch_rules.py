"""The launch rules that depend on sizes alone (csrc/shape_launch.hpp), built
for the host and checked at sizes no test would launch: a launch holds fewer
than 2^32 work-items along x, or the runtime refuses it."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_20766_amd", "csrc")
SHIM = """
#include "shape_launch.hpp"
using namespace shape;
extern "C" {
int64_t r_max_workgroups(int threads) { return max_workgroups(threads); }
int r_align_waves(int64_t pairs, int starts, int fit, int crowded, int n_cu) {
  return align_waves(pairs, starts, fit, crowded, n_cu);
}
int r_align_splits_starts(int64_t pairs, int starts, int steps, int busy, int resident,
                          double mean_b, int n_cu) {
  return align_splits_starts(pairs, starts, steps, busy, resident, mean_b, n_cu);
}
int r_align_starts_per_block(int64_t pairs, int starts, int waves, int n_cu) {
  return align_starts_per_block(pairs, starts, waves, n_cu);
}
int r_prepare_apart(int64_t blocks, int a, int b) { return prepare_apart(blocks, a, b); }
int r_align_split_fits(int64_t dynamic, int64_t own, int64_t max_lds) {
  return align_split_fits(dynamic, own, max_lds);
}
int r_screen_shape(int adaptive, int seeded, int64_t pairs, int64_t rounds, double expected,
                   int side, int64_t lds, int n_cu, int* first) {
  const ScreenShape s = screen_shape(adaptive, seeded, pairs, rounds, expected, side, lds, n_cu);
  *first = s.first;
  return s.rounds;
}
double r_expected(double tau, int side, double q, double b) {
  return screen_rounds_expected(tau, side, q, b);
}
}
"""
LIMIT = 1 << 32


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(SHIM)
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    L.r_max_workgroups.restype = ctypes.c_int64
    L.r_align_waves.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
    L.r_align_splits_starts.argtypes = ([ctypes.c_int64] + [ctypes.c_int] * 4 +
                                        [ctypes.c_double, ctypes.c_int])
    L.r_align_starts_per_block.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3
    L.r_prepare_apart.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    L.r_align_split_fits.argtypes = [ctypes.c_int64] * 3
    L.r_screen_shape.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64,
                                 ctypes.c_double, ctypes.c_int, ctypes.c_int64, ctypes.c_int,
                                 ctypes.POINTER(ctypes.c_int)]
    L.r_expected.argtypes = [ctypes.c_double, ctypes.c_int, ctypes.c_double, ctypes.c_double]
    L.r_expected.restype = ctypes.c_double
    return L


@pytest.mark.parametrize("threads", [64, 128, 256, 512, 1024])
def test_a_launch_stays_below_the_work_item_limit(rules, threads):
    n = rules.r_max_workgroups(threads)
    assert n * threads < LIMIT <= (n + 1) * threads


@pytest.mark.parametrize("pairs", [1, 255, 256, 4096, (1 << 23) - 1, 1 << 23, (1 << 24) - 1])
@pytest.mark.parametrize("starts", [1, 7, 8, 16, 1000])
def test_alignment_workgroups_fit_a_launch(rules, pairs, starts):
    """Up to 2^24 - 1 pairs, as with four waves per workgroup throughout."""
    for crowded in (0, 1):
        waves = rules.r_align_waves(pairs, starts, 1, crowded, 256)
        assert waves in (4, 8) and pairs * waves * 64 < LIMIT
        assert rules.r_align_waves(pairs, starts, 0, crowded, 256) == 4


@pytest.mark.parametrize("pairs", [1, 7168, 12800, 12801, (1 << 24) - 1, 1 << 24, (1 << 25) - 1,
                                   1 << 25, (1 << 26) - 1])
@pytest.mark.parametrize("lds", [2000, 6400, 8000, 16000, 24000])  # bytes per pair
@pytest.mark.parametrize("adaptive,side,rounds", [(0, 256, 16), (0, 64, 1), (1, 256, 128),
                                                  (1, 4096, 8), (1, 64, 2)])
def test_screen_workgroups_fit_a_launch(rules, pairs, lds, adaptive, side, rounds):
    """Up to 2^26 - 1 pairs, as with one wave per pair throughout, however
    much LDS a pair takes."""
    first = ctypes.c_int()
    for expected, seeded in ((0.1, 0), (5.0, 0), (50.0, 0), (0.1, 1), (50.0, 1)):
        R = rules.r_screen_shape(adaptive, seeded, pairs, rounds, expected, side, lds, 256,
                                 ctypes.byref(first))
        assert R in (1, 2, 4) and R <= rounds and pairs * R * 64 < LIMIT
        assert first.value == R if not adaptive else 1 <= first.value <= R


def test_a_kernels_own_lds_counts_towards_the_limit(rules):
    most = 160 * 1024
    assert rules.r_align_split_fits(most - 80, 72, most)
    assert not rules.r_align_split_fits(most - 64, 72, most)
    assert not rules.r_align_split_fits(most, 72, most)


def test_starts_run_by_themselves_only_where_their_waves_have_samples(rules):
    split = rules.r_align_splits_starts
    # 10 and 100 pairs x 16 starts of 2,048 samples; not 500 x 4 of 256
    assert split(10, 16, 60, 16, 16, 30.0, 256) and split(100, 16, 60, 16, 16, 30.0, 256)
    assert not split(500, 4, 8, 2, 32, 30.0, 256) and not split(250, 8, 8, 4, 32, 30.0, 256)
    assert not split(1000, 1, 0, 2, 9, 30.0, 256)
    # nor small molecules, but for a handful
    assert split(10, 16, 60, 16, 16, 5.0, 256) and not split(100, 16, 60, 16, 16, 5.0, 256)
    assert split(20000, 1, 8, 16, 4, 30.0, 256) and not split(20000, 1, 8, 16, 4, 5.0, 256)
    # never more workgroups than a launch holds
    for pairs in (1, 1 << 22, (1 << 22) - 1, 1 << 31):
        for resident in (1, 4, 16):
            if split(pairs, 1, 8, 16, resident, 30.0, 256):
                assert pairs * 1024 < LIMIT


@pytest.mark.parametrize("pairs", [1, 300, 767, 768, 2047, 2048, 1 << 23])
@pytest.mark.parametrize("starts", [1, 3, 4, 8, 9, 20, 65535, 65536, 600000])
def test_starts_of_a_pair_are_covered_by_a_grid(rules, pairs, starts):
    for waves in (4, 8):
        spb = rules.r_align_starts_per_block(pairs, starts, waves, 256)
        assert spb >= 1 and (starts + spb - 1) // spb <= 65535


def test_eight_waves_only_where_the_last_eight_starts_fill_most_of_them(rules):
    waves = [rules.r_align_waves(5000, s, 1, 0, 256) for s in range(1, 26)]
    assert waves == [4] * 7 + [8] + [4] * 4 + [8] * 4 + [4] * 4 + [8] * 4 + [4]


def test_pairs_that_need_one_round_get_one_wave(rules):
    """Adaptive screens at a coarse tau, fewer pairs than fill the chip."""
    first = ctypes.c_int()

    def R(pairs, tau, atoms):
        e = rules.r_expected(tau, 256, 30.0, atoms)
        return rules.r_screen_shape(1, 0, pairs, 128, e, 256, 4000, 256, ctypes.byref(first))

    for pairs in (1000, 3000, 7000, 12500):
        assert R(pairs, 0.05, 30.0) == 1, pairs
        # half of them a second round: together where the chip has waves to spare
        assert R(pairs, 0.02, 30.0) == (2 if pairs == 1000 else 1), pairs
        assert R(pairs, 0.005, 30.0) > 1 and R(pairs, 0.01, 2.5) == 1, pairs


def test_large_molecules_that_need_a_few_rounds_get_them_together(rules):
    """As many in the first pass as their pairs take, where LDS holds few pairs."""
    first = ctypes.c_int()

    def shape(pairs, expected, lds):
        return rules.r_screen_shape(1, 0, pairs, 128, expected, 256, lds, 256,
                                    ctypes.byref(first)), first.value

    assert shape(9000, 4.4, 9600) == (2, 2) and shape(9000, 2.2, 9600) == (2, 2)
    assert shape(9000, 1.1, 9600) == (2, 1) and shape(800, 1.1, 9600) == (2, 2)
    assert shape(9000, 4.4, 24000) == (4, 4) and shape(9000, 2.2, 24000) == (4, 2)
    assert shape(9000, 1.1, 24000) == (2, 1)


@pytest.mark.parametrize("seeded", [0, 1])
def test_pairs_whose_tau_needs_many_rounds_get_whole_passes(rules, seeded):
    """Budgets add to what tau asks for."""
    first = ctypes.c_int()
    for pairs, expected in ((1000, 17.0), (2336, 4.7), (3584, 4.0), (3585, 8.0), (12800, 17.0)):
        R = rules.r_screen_shape(1, seeded, pairs, 128, expected, 256, 4000, 256,
                                 ctypes.byref(first))
        assert first.value == R > 1, pairs


def test_sets_are_prepared_apart_only_if_that_leaves_less_in_a_launch(rules):
    most = rules.r_max_workgroups(256)
    assert not rules.r_prepare_apart(most, 1, 1 << 26)
    assert rules.r_prepare_apart(most + 1, 1, 1 << 26)
    # one set alone is left to the runtime's refusal
    assert not rules.r_prepare_apart(most + 1, 1 << 27, 0)
    assert not rules.r_prepare_apart(most + 1, 0, 1 << 27)
