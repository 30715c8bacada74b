"""The fused network's tile sizes.

The rows per tile follow from the number of atoms (and, for BF16, of ensemble
members).  A row's result does not depend on the tile it sits in, so in the
deterministic mode a molecule's energy and forces are the same bits in a call
small enough for 16-row tiles, in one for 32-row tiles and in one for the
largest, with and without gradients; and the small call is held to the oracle.
The molecules leave groups of one row, of a few, and of several tiles and a
remainder.
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import check_forces, potential, to_dev
from paper_2310_03121_amd import Potential

pytestmark = pytest.mark.gpu

SMALL, MIDDLE, LARGE = 6, 110, 300   # molecules: 249, 4,581 and 12,432 atoms


@pytest.mark.parametrize("members", [1, 3])
@pytest.mark.parametrize("S", [4, 7])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_tiles_agree_bit_for_bit(prec, S, members):
    sizes = [1, 2, 17, 64, 65, 100] + [10 + (37 * k) % 64 for k in range(LARGE - SMALL)]
    mols = [w.single_molecule(n, seed=900 + k, n_species=S) for k, n in enumerate(sizes)]
    at = w.aev_table(S)
    mts = [w.mlp_table(S, seed=50 + k) for k in range(members)]
    pot = Potential.ensemble_from_tables(at, mts, precision=prec, max_neighbors=64,
                                         deterministic=True)
    ref = None
    for k in (LARGE, MIDDLE, SMALL):
        s = w.pack_molecules(mols[:k], S)
        print(f"\n[case] {prec} S={S} members={members} N={s.n_atoms}", flush=True)
        pos, sp, off = to_dev(s)
        E, F = pot.energy_forces(pos, sp, off)
        pot.check()
        E0, _ = pot.energy_forces(pos, sp, off, forces=False)
        pot.check()
        if ref is None:
            ref = (E, F, E0)
        assert torch.equal(E, ref[0][:k])
        assert torch.equal(F, ref[1][:s.n_atoms])
        assert torch.equal(E0, ref[2][:k])
    r = o.ensemble_energy_forces(s, aev_table=at, mlp_tables=mts)
    check_forces(F.cpu().numpy(), r.F, prec, f"tiles S={S} members={members}")
    scale = max(np.abs(r.E_atom).sum() / s.n_mol, np.abs(r.E_atom).mean())
    bar = 1e-5 if prec == "fp32" else 1e-2
    for e in (E, E0):
        assert np.abs(e.cpu().numpy() - r.E).max() <= bar * scale
