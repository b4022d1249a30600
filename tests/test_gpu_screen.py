"""GPU parity of screening (shape_screen) against the FP64 oracle on identical
samples: fixed budgets and confidence-bounded adaptive rounds, small
libraries in full and the 100,000-molecule library on sampled pairs."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2607_20766_amd import molgen
from paper_2607_20766_amd.engine import (Engine, LAMBDA_P27, SHAPE_SCREEN_ADAPTIVE,
                                         SHAPE_SCREEN_FIXED, ShapeError)
from tests.gpu_common import (compare_adaptive, compare_screen, oracle_mol, rel_err,
                              require_gpu)

pytestmark = pytest.mark.gpu

QUERY_ID = 0xFFFFFF00


@pytest.fixture(scope="module")
def eng():
    require_gpu()
    return Engine(0)


@pytest.fixture(scope="module")
def small_lib():
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(11, 61, 10, 50, workers=1)  # ragged: not a multiple of 4 waves
    return q, L


def _oracle_screen(q, L, **kw):
    la = O.alpha_from_radius(L.radius, LAMBDA_P27)
    return O.screen(oracle_mol(O, q), QUERY_ID, L.offsets, L.xyz, la, **kw)


def _to_np(out):
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("n_side", [4096, 320])
def test_fixed_small_library(eng, small_lib, n_side):
    q, L = small_lib
    print(f"case: fixed screen, 61 molecules, n_side={n_side}", flush=True)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_FIXED, n_per_side=n_side, seed=7))
    torch.cuda.synchronize()
    r = _oracle_screen(q, L, mode=0, n_fixed=n_side, seed=7)
    compare_screen(g, r)
    assert np.all(g["n_used"] == 2 * n_side)


def test_fixed_pair_subset_and_self(eng, small_lib):
    q, L = small_lib
    # put the query itself into the library with the query's stream id
    Lq = molgen.MolSet.concat([L, q])
    ids = np.arange(Lq.n_mols, dtype=np.uint32)
    ids[-1] = QUERY_ID
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(Lq, mol_id=ids)
    pairs = torch.tensor([Lq.n_mols - 1, 5, 5, 0, 60], dtype=torch.int32, device="cuda")
    g = _to_np(eng.shape_screen(Q, lib, n_per_side=1024, seed=2, pairs=pairs))
    assert g["T"][0] == 1.0
    assert g["T"][1] == g["T"][2]
    la = O.alpha_from_radius(Lq.radius, LAMBDA_P27)
    r = O.screen(oracle_mol(O, q), QUERY_ID, Lq.offsets, Lq.xyz, la, lib_id=ids,
                 pairs=pairs.cpu().numpy(), mode=0, n_fixed=1024, seed=2)
    compare_screen(g, r)


def test_adaptive_small_library(eng, small_lib):
    q, L = small_lib
    tau, cap = 0.005, 65536
    print("case: adaptive screen, 61 molecules, tau=0.005", flush=True)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512,
                                cap_per_pair=cap, tau=tau, seed=1))
    r = _oracle_screen(q, L, mode=1, round_per_pair=512, cap_per_pair=cap, tau=tau, seed=1)
    compare_adaptive(g, r, q, L, tau, cap, 1, QUERY_ID, min_same=0.95)
    assert np.all(g["n_used"] % 512 == 0)


def test_adaptive_tiny_and_huge_tau(eng, small_lib):
    q, L = small_lib
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512,
                                cap_per_pair=2048, tau=1e-9, seed=1))
    assert np.all(g["n_used"] == 2048)
    g = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512,
                                cap_per_pair=2048, tau=1e9, seed=1))
    assert np.all(g["n_used"] == 512)
    f = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_FIXED, n_per_side=256, seed=1))
    assert np.array_equal(g["T"], f["T"])  # one adaptive round == fixed 256 per side


def test_full_library_sampled_pairs(eng):
    """The 100,000-molecule screen: 30-atom query vs 100,000 molecules (10-50 atoms),
    4096 samples per side; 96 pairs spread over the library checked against
    the oracle one by one."""
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(1, 100000, 10, 50)
    print("case: full 100k library fixed 4096", flush=True)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, n_per_side=4096, seed=0))
    assert np.all(np.isfinite(g["T"]))
    idx = np.unique(np.concatenate([np.arange(8), np.arange(99992, 100000),
                                    np.random.default_rng(0).integers(0, 100000, 80)]))
    r = _oracle_screen(q, L, pairs=idx.astype(np.int32), mode=0, n_fixed=4096, seed=0)
    compare_screen({k: v[idx] for k, v in g.items()}, r)
    # repeatable bit for bit
    g2 = _to_np(eng.shape_screen(Q, lib, n_per_side=4096, seed=0))
    for k in g:
        assert np.array_equal(g[k], g2[k])


def test_full_library_adaptive_sampled_pairs(eng):
    """The headline confidence-bounded screen in the launch configuration the
    benchmark times (autotuned tile, one 64-lane workgroup per pair, 100,000
    workgroups renumbered in tiles of 64 pairs per XCD): tau 0.005, rounds of
    512, cap 65,536; 96 pairs spread over the library (both ends, the
    neighbourhood of the first tile boundaries, random) against the oracle."""
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(1, 100000, 10, 50)
    tau, cap = 0.005, 65536
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=cap, tau=tau, seed=0)
    print("case: full 100k library adaptive, tuned tile", flush=True)
    eng.shape_screen_tune(Q, lib, **kw)
    g = _to_np(eng.shape_screen(Q, lib, **kw))
    eng.screen_variant(-1)
    assert np.all(np.isfinite(g["T"]))
    assert np.all((g["se_T"] <= tau * (1 + 1e-6)) | (g["n_used"] == cap))
    idx = np.unique(np.concatenate([np.arange(6), np.arange(60, 70), np.arange(508, 516),
                                    np.arange(99994, 100000),
                                    np.random.default_rng(5).integers(0, 100000, 66)]))
    assert idx.size >= 96
    r = _oracle_screen(q, L, pairs=idx.astype(np.int32), mode=1, round_per_pair=512,
                       cap_per_pair=cap, tau=tau, seed=0)
    compare_adaptive(g, r, q, L, tau, cap, 0, QUERY_ID, idx=idx)


def test_invalid_molecules_flagged(eng, small_lib):
    q, L = small_lib
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    lib.alpha[int(L.offsets[4])] = -1.0
    g = _to_np(eng.shape_screen(Q, lib, n_per_side=256, seed=0))
    assert np.isnan(g["T"][4]) and np.all(np.isfinite(np.delete(g["T"], 4)))
    with pytest.raises(ShapeError) as e:
        eng.shape_check_data()
    assert e.value.code == -6
    eng.shape_check_data()  # flag cleared
    with pytest.raises(ShapeError):
        eng.shape_screen(Q, lib, n_per_side=100)
    out = eng.shape_screen(Q, lib, n_per_side=256, n_pairs=0)
    assert out["T"].numel() == 0


@pytest.mark.parametrize("q_atoms", [1, 256])
def test_extreme_sizes_every_tile_variant(eng, q_atoms):
    """1- and 256-atom molecules (the minimum and SHAPE_MAX_ATOMS) on both
    sides, sizes around the 64-lane width, every tile variant of the
    screening kernel, adaptive rounds: identical across variants and equal to
    the oracle."""
    from paper_2607_20766_amd.engine import SHAPE_SCREEN_VARIANTS
    q = molgen.molecule(3, 1, q_atoms)
    L = molgen.MolSet.concat([molgen.molecule(4, i, n)
                              for i, n in enumerate((1, 2, 63, 64, 65, 256, 7, 128))])
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=4096, tau=0.005,
              seed=6)
    print(f"case: extreme sizes, query {q_atoms} atoms", flush=True)
    ref = None
    for v in range(SHAPE_SCREEN_VARIANTS):
        eng.screen_variant(v)
        g = _to_np(eng.shape_screen(Q, lib, **kw))
        if ref is None:
            ref = g
        for k in g:
            assert np.array_equal(g[k], ref[k]), (v, k)
    eng.screen_variant(-1)
    r = _oracle_screen(q, L, mode=1, round_per_pair=512, cap_per_pair=4096, tau=0.005, seed=6)
    compare_adaptive(ref, r, q, L, 0.005, 4096, 6, QUERY_ID, min_same=0.75)


def test_odd_atom_counts(eng):
    """Odd query and library sizes (LDS arrays of 8-byte records after odd
    counts of 4-byte ones must stay aligned)."""
    q = molgen.molecule(1, 5, 31)
    L = molgen.library(12, 9, 11, 17, workers=1)
    assert int(L.sizes().max()) % 2 == 1 or q.n_atoms % 2 == 1
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, n_per_side=512, seed=4))
    r = _oracle_screen(q, L, mode=0, n_fixed=512, seed=4)
    compare_screen(g, r)


def test_adaptive_seeded_budgets(eng, small_lib):
    """Per-pair budgets defer the first stop test; GPU and oracle agree."""
    q, L = small_lib
    rng = np.random.default_rng(8)
    n_start = (rng.integers(1, 40, L.n_mols) * 512).astype(np.int32)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    g = _to_np(eng.shape_screen(Q, lib, mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512,
                                cap_per_pair=16384, tau=0.005, seed=3,
                                n_start=torch.from_numpy(n_start).cuda()))
    r = _oracle_screen(q, L, mode=1, round_per_pair=512, cap_per_pair=16384, tau=0.005,
                       seed=3, n_start=n_start)
    assert np.all(g["n_used"] >= np.minimum(n_start, 16384))
    compare_adaptive(g, r, q, L, 0.005, 16384, 3, QUERY_ID, min_same=0.95)


def test_screen_resumes_from_checkpoint(eng, tmp_path):
    """An adaptive screen run in chunks of pairs, interrupted after two
    chunks and resumed from its state file, equals one whole-library screen
    bit for bit; a state file of another screen is refused."""
    from paper_2607_20766_amd.resume import screen_in_chunks
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(23, 1000, 10, 50, workers=1)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=8192, tau=0.005,
              seed=8)
    full = _to_np(eng.shape_screen(Q, lib, **kw))
    path = str(tmp_path / "screen.safetensors")
    print("case: chunked screen, interrupted after two chunks", flush=True)
    assert screen_in_chunks(eng, Q, lib, 300, path, stop_after=2, **kw) is None
    out = screen_in_chunks(eng, Q, lib, 300, path, **kw)
    for k in full:
        assert np.array_equal(out[k], full[k]), k
    with pytest.raises(ValueError):
        screen_in_chunks(eng, Q, lib, 300, path, **dict(kw, seed=9))


def test_allocation_failure_is_reported_and_recovered(eng):
    """Injected out-of-memory failures of a fresh context's scratch (one,
    then three calls in a row) come back as SHAPE_E_NOMEM without a launch
    that could use the missing buffer; the same context then screens
    normally, to the bits of another context."""
    from paper_2607_20766_amd.engine import ShapeError
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(24, 300, 10, 50, workers=1)
    Q = eng.molecules(q, mol_id=[QUERY_ID])
    lib = eng.molecules(L)
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=8192, seed=2)
    want = _to_np(eng.shape_screen(Q, lib, **kw))
    for n_fail in (1, 3):
        e2 = Engine(0)
        e2.fail_allocations(n_fail)
        print(f"case: {n_fail} injected allocation failures", flush=True)
        for _ in range(n_fail):
            with pytest.raises(ShapeError) as err:
                e2.shape_screen(Q, lib, **kw)
            assert err.value.code == -3
        got = _to_np(e2.shape_screen(Q, lib, **kw))
        for k in want:
            assert np.array_equal(got[k], want[k]), k
    with pytest.raises(ShapeError):
        eng.fail_allocations(-1)


@pytest.mark.parametrize("case", ["fixed", "adaptive", "seeded", "antithetic"])
def test_long_screen_in_launch_order_same_bits(case):
    """A screen of at least 16 pairs per compute unit runs its pairs longest
    first (the order comes from the atom counts and any seeded budgets);
    every pair's outputs equal those of the same pair screened in calls of
    1,000 pairs, which keep the plain order, bit for bit.  The pairs repeat
    molecules, mix 1- to 96-atom molecules and include indices outside the
    library (NaN, no samples)."""
    require_gpu()
    e = Engine(0)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 16 * n_cu + 123
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(26, 2500, 1, 96, workers=4)
    rng = np.random.default_rng(26)
    pairs = rng.integers(0, L.n_mols, n).astype(np.int32)
    pairs[rng.choice(n, 9, replace=False)] = [-1, -7, L.n_mols, L.n_mols + 3, -1, L.n_mols,
                                              -2, L.n_mols + 1, -1]
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=4096, tau=0.01,
              seed=5)
    if case == "fixed":
        kw = dict(mode=SHAPE_SCREEN_FIXED, n_per_side=256, seed=5)
    n_start = None
    if case == "seeded":
        n_start = (rng.integers(0, 9, n) * 512).astype(np.int32)
    e.sampling(case == "antithetic")
    Q = e.molecules(q, mol_id=[QUERY_ID])
    lib = e.molecules(L)
    dev = e.torch_device
    print(f"case: {case}, {n} pairs", flush=True)
    full = _to_np(e.shape_screen(
        Q, lib, pairs=torch.from_numpy(pairs).to(dev),
        n_start=None if n_start is None else torch.from_numpy(n_start).to(dev), **kw))
    parts = []
    for a in range(0, n, 1000):
        sl = slice(a, min(n, a + 1000))
        parts.append(_to_np(e.shape_screen(
            Q, lib, pairs=torch.from_numpy(pairs[sl]).to(dev),
            n_start=None if n_start is None else torch.from_numpy(n_start[sl]).to(dev), **kw)))
    e.sampling(False)
    bad = (pairs < 0) | (pairs >= L.n_mols)
    for k in full:
        got = np.concatenate([p[k] for p in parts])
        assert np.array_equal(full[k], got, equal_nan=k != "n_used"), k
    assert np.all(np.isnan(full["T"][bad])) and np.all(full["n_used"][bad] == 0)
    assert np.all(np.isfinite(full["T"][~bad]))


def test_long_screen_order_edge_cases():
    """The launch order at its threshold (exactly 16 pairs per compute unit)
    with budgets below zero, zero and far above the cap, against calls too
    small to be reordered, bit for bit; and a long screen whose pairs all lie
    outside the library (every output NaN, no samples)."""
    require_gpu()
    e = Engine(0)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 16 * n_cu
    q = molgen.molecule(1, 0, 30)
    L = molgen.library(28, 1500, 5, 60, workers=4)
    Q, lib = e.molecules(q, mol_id=[QUERY_ID]), e.molecules(L)
    dev = e.torch_device
    rng = np.random.default_rng(28)
    pairs = rng.integers(0, L.n_mols, n).astype(np.int32)
    n_start = rng.choice(np.array([-5, 0, 512, 3000, 10**9], np.int32), n)
    kw = dict(mode=SHAPE_SCREEN_ADAPTIVE, round_per_pair=512, cap_per_pair=4096, tau=0.01,
              seed=8)
    print(f"case: {n} pairs at the threshold, extreme budgets", flush=True)
    full = _to_np(e.shape_screen(Q, lib, pairs=torch.from_numpy(pairs).to(dev),
                                 n_start=torch.from_numpy(n_start).to(dev), **kw))
    parts = []
    for a in range(0, n, 777):
        sl = slice(a, min(n, a + 777))
        parts.append(_to_np(e.shape_screen(Q, lib, pairs=torch.from_numpy(pairs[sl]).to(dev),
                                           n_start=torch.from_numpy(n_start[sl]).to(dev),
                                           **kw)))
    for k in full:
        assert np.array_equal(full[k], np.concatenate([p[k] for p in parts])), k
    assert np.all(full["n_used"][n_start >= 4096] == 4096)
    print("case: a long screen of pairs outside the library", flush=True)
    bad = torch.full((n + 5,), -1, dtype=torch.int32, device=dev)
    bad[::2] = L.n_mols
    out = _to_np(e.shape_screen(Q, lib, pairs=bad, **kw))
    assert np.all(np.isnan(out["T"])) and np.all(out["n_used"] == 0)


@pytest.mark.parametrize("variant", [-1, 0, 1, 3, 6])
def test_points_whose_squared_norm_overflows(eng, variant):
    """A query so wide (alpha 2e-38, sd 5e18) that |r|^2 of some of its samples
    is beyond FP32: every occupancy is 0 there, for libraries of odd and of
    even molecules."""
    print(f"case: overflowing squared norms, variant {variant}", flush=True)
    Q = eng.molecules(molgen.molecule(12, 0, 1), mol_id=[QUERY_ID])
    Q.alpha.fill_(2e-38)
    lib = eng.molecules(molgen.MolSet.concat([molgen.molecule(12, n, n)
                                              for n in (1, 2, 3, 4, 9)]))
    eng.screen_variant(variant)
    try:
        g = _to_np(eng.shape_screen(Q, lib, n_per_side=4096, seed=7))
    finally:
        eng.screen_variant(-1)
    for k in ("T", "se_T", "O_ab", "O_bb"):
        assert np.all(np.isfinite(g[k])), (k, g[k])
    # O_AA is about 10^56 times O_AB
    assert np.all(np.abs(g["T"]) < 1e-30) and np.all(g["O_ab"] >= 0)
