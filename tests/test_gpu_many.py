"""Calls over millions of tiny molecules, beyond what one launch of wide
workgroups holds: the same values as a small call of the same molecules."""
import pytest
import torch

from paper_2607_20766_amd import molgen
from paper_2607_20766_amd.engine import Engine, Molecules
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu
PERIOD = 1009


@pytest.fixture(scope="module")
def eng():
    require_gpu()
    return Engine(0)


def _atoms(eng, n, shift=0.0):
    """n one-atom molecules, repeating every PERIOD (ids too)."""
    dev = eng.torch_device
    i = torch.arange(n, device=dev, dtype=torch.int32) % PERIOD
    x = i.to(torch.float32)
    xyz = torch.stack([0.001 * x + shift, 0.002 * x, -0.001 * x], 1).contiguous()
    return Molecules(torch.arange(n + 1, device=dev, dtype=torch.int32), xyz,
                     (0.5 + 0.001 * x).contiguous(), i.contiguous(), 1)


def _repeats(big, small):
    n = big.shape[0]
    whole = n // PERIOD * PERIOD
    assert torch.equal(big[:whole].reshape(whole // PERIOD, *small.shape),
                       small.expand(whole // PERIOD, *small.shape))
    assert torch.equal(big[whole:], small[:n - whole])


def test_self_overlap_of_over_four_million_molecules(eng):
    n = (1 << 22) + 5
    print(f"case: self-overlap of {n} molecules", flush=True)
    ref = eng.shape_self_overlap(_atoms(eng, PERIOD), 64, seed=5)
    got = eng.shape_self_overlap(_atoms(eng, n), 64, seed=5)
    assert torch.isfinite(ref).all()
    _repeats(got, ref)


def test_alignment_of_over_two_million_pairs(eng):
    n = (1 << 21) + 3
    print(f"case: alignment of {n} pairs", flush=True)
    pose = torch.zeros(n, 1, 7, device=eng.torch_device)
    pose[:, :, 0] = 1.0
    small = pose[:PERIOD].clone()
    T_ref, _ = eng.shape_align(_atoms(eng, PERIOD), _atoms(eng, PERIOD, 0.3), small, 64, 1, seed=5)
    T, _ = eng.shape_align(_atoms(eng, n), _atoms(eng, n, 0.3), pose, 64, 1, seed=5)
    assert torch.isfinite(T_ref).all()
    _repeats(T, T_ref)
    _repeats(pose, small)


def test_screen_of_over_sixteen_million_pairs_of_a_large_molecule_library(eng):
    """A library whose largest molecule (200 atoms) asks for several waves per
    pair; the list holds 2^24 + 9 pairs."""
    n = (1 << 24) + 9
    print(f"case: screen of {n} listed pairs", flush=True)
    q = eng.molecules(molgen.molecule(91, 0, 3), mol_id=[7])
    L = eng.molecules(molgen.MolSet.concat(
        [molgen.molecule(91, 1, 200)] + [molgen.molecule(91, i, 2) for i in range(2, PERIOD)]))
    ref = eng.shape_screen(q, L, n_per_side=320, seed=5)
    # the large molecule once, then the small ones in turn
    pairs = 1 + torch.arange(n, device=eng.torch_device, dtype=torch.int32) % (PERIOD - 2)
    pairs[-1] = 0
    out = {k: torch.empty(n, device=eng.torch_device) for k in ("T", "se_T")}
    eng.shape_screen(q, L, n_per_side=320, seed=5, pairs=pairs, out=out)
    for k, v in out.items():
        assert torch.equal(v, ref[k][pairs.long()])
