"""The molecule pair scan with four atoms per wave, and the species sort's two
forms.

Molecules of sizes around a wave (64), around the candidates that stay in
registers (192) and below a wave's four atoms, in an order that puts their
boundaries at every place of a wave; the pair sets are those of the float32
predicate exactly, one atom below, at and above the size that switches.  Beyond
131,072 atoms the sort takes launches of its own; in the deterministic mode the
energies and forces are the bits of the same molecules in smaller calls.
"""
import numpy as np
import pytest
import torch

import workloads as w
from gpu_util import pair_set_from_ell, potential, to_dev
from oracle.neighbors import pair_list

pytestmark = pytest.mark.gpu


def _batch(n):
    """n atoms of seven elements in molecules of many sizes."""
    sizes = [1, 2, 3, 5, 63, 64, 65, 127, 129, 191, 192, 193, 250]
    mols, left, k = [], n, 0
    while left:
        m = min(sizes[k % len(sizes)], left)
        mols.append(w.single_molecule(m, seed=300 + k % 40, n_species=7))
        left -= m
        k += 1
    return w.pack_molecules(mols, 7)


@pytest.mark.parametrize("n", [16383, 16384, 16385, 20001])
def test_pairs_of_ragged_molecules(n):
    s = _batch(n)
    print(f"\n[case] ragged molecules N={n}", flush=True)
    pot, at, _ = potential(7, "fp32", max_neighbors=128)
    pos, sp, off = to_dev(s)
    pot.energy_forces(pos, sp, off)
    pot.check()
    counts, nbr = pot.debug_neighbors(n)
    I, J = pair_set_from_ell(counts, nbr)
    Io, Jo = pair_list(s.pos, s.mol_offsets, None, at.rc_rad)
    assert np.array_equal(I, Io) and np.array_equal(J, Jo)


def test_sort_beyond_the_fused_limit():
    mols, part = 2060, 515  # 131,840 and 32,960 atoms
    s = w.conformer_batch(mols, 64, seed=1)
    print(f"\n[case] N={s.n_atoms}", flush=True)
    pot, _, _ = potential(7, "bf16", max_neighbors=64, deterministic=True)
    pos, sp, off = to_dev(s)
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    o1 = off[:part + 1].contiguous()
    for m in range(0, mols, part):
        a, b = 64 * m, 64 * (m + part)
        E1, F1 = pot.energy_forces(pos[a:b].contiguous(), sp[a:b].contiguous(), o1)
        pot.check()
        assert torch.equal(E1, E[m:m + part])
        assert torch.equal(F1, F[a:b])
