"""Calls with less to do take accordingly less time: launch shapes chosen for
large calls must not be forced on small ones.  Ratios of times on one box, with
room for noise; what a wrong shape costs is stated at each test."""
import time

import numpy as np
import pytest
import torch

from paper_2607_20766_amd import molgen
from paper_2607_20766_amd.engine import SHAPE_SCREEN_ADAPTIVE, Engine
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    require_gpu()
    return Engine(0)


@pytest.fixture(scope="module")
def base():
    return molgen.library(93, 400, 10, 50, workers=4)


def _library(eng, base, n):
    return eng.molecules(base.subset(np.arange(n) % base.n_mols))


def _ms(f, repeat=5):
    f()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(repeat):
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return 1e3 * best


def _kernel_ms(eng, f, repeat=9):
    """The best time of f's screening kernel, by HIP events."""
    eng.shape_timing_enable()
    try:
        f()
        best = 1e9
        for _ in range(repeat):
            eng.shape_timing_read()
            f()
            best = min(best, eng.shape_timing_read()[0])
    finally:
        eng.shape_timing_enable(False)
    return best


def test_self_overlap_of_few_samples(eng, base):
    """1/32 of the samples; in workgroups of 1,024 threads 0.68 of the time."""
    M = _library(eng, base, 100_000)
    few, many = (_ms(lambda: eng.shape_self_overlap(M, n, seed=1)) for n in (64, 2048))
    print(f"case: 100,000 self-overlaps, 64 samples {few:.3f} ms, 2,048 {many:.3f}", flush=True)
    assert few < 0.4 * many


def test_alignment_of_few_samples(eng, base):
    """1/8 of the samples; with sixteen waves per start, most without a sample,
    half of the time (369 against 720 us)."""
    A, B = _library(eng, base, 500), eng.molecules(base.subset((np.arange(500) * 7 + 3) % 400))
    pose = torch.zeros(500, 4, 7, device=eng.torch_device)
    pose[:, :, 0] = 1.0
    few, many = (_ms(lambda: eng.shape_align(A, B, pose.clone(), n, 8, seed=1))
                 for n in (256, 2048))
    print(f"case: 500 x 4 alignments, 256 samples {few:.3f} ms, 2,048 {many:.3f}", flush=True)
    assert few < 0.35 * many


def test_alignment_starts_of_many_pairs_of_large_molecules(eng):
    """20 times the pairs; with the atoms in LDS, eight pairs of one wave in
    a compute unit's, 19 times the time (67 against 1,300 us)."""
    lib = molgen.library(94, 60, 150, 256, workers=4)
    q = eng.molecules(molgen.molecule(94, 100, 30), mol_id=[1])
    L = [_library(eng, lib, n) for n in (2000, 40_000)]
    few, many = (_ms(lambda: eng.shape_fo_starts(q, M, 3, seed=1)) for M in L)
    print(f"case: starts, 2,000 pairs {few:.3f} ms, 40,000 {many:.3f}", flush=True)
    assert many < 9 * few


def test_screens_of_short_rounds(eng, base):
    """The same samples in rounds of 128 per side, two per lane, instead of 256;
    with tiles of four points, half of them unused, twice the time."""
    lib = _library(eng, base, 20_000)
    q = eng.molecules(molgen.molecule(94, 1, 30), mol_id=[1])
    short, whole = (_kernel_ms(eng, lambda: eng.shape_screen(
        q, lib, mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=r, cap_per_pair=8192, tau=0.001,
        seed=1)) for r in (256, 512))
    print(f"case: 20,000 pairs, rounds of 128 {short:.3f} ms, of 256 {whole:.3f}", flush=True)
    assert short < 1.4 * whole


def test_screens_that_stop_in_their_first_round(eng, base):
    """Pairs of one round each (tau 0.05), 7,000 of them: with four rounds of
    every pair drawn at once 1.6 times the time of one wave per pair."""
    lib = _library(eng, base, 7000)
    q = eng.molecules(molgen.molecule(94, 1, 30), mol_id=[1])
    ms = {}
    for variant in (-1, 3):  # the library's choice, one wave per pair
        eng.screen_variant(variant)
        ms[variant] = _kernel_ms(eng, lambda: eng.shape_screen(
            q, lib, mode=SHAPE_SCREEN_ADAPTIVE, tau=0.05, seed=1))
    eng.screen_variant(-1)
    print(f"case: 7,000 pairs, tau 0.05, {ms[-1]:.3f} ms, one wave {ms[3]:.3f}", flush=True)
    assert ms[-1] < 1.25 * ms[3]
