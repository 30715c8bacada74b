"""An FP32 ensemble's dE/dG on both sides of 1,024 atoms.

Up to there it runs in 16-row tiles whose deltas lie in LDS, above in 64-row
tiles that stream them; the sums are the same, so in the deterministic mode the
forces of the molecules that both calls hold are the same bits.  Two and eight
members of 160 and 256 columns give products of 20 to 128 steps, whole rings of
16 and remainders; the molecules leave tiles of one row and of several.
"""
import pytest
import torch

import workloads as w
from gpu_util import to_dev
from paper_2310_03121_amd import Potential

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [2, 8])
@pytest.mark.parametrize("S", [4, 7])
def test_both_forms_agree_bit_for_bit(S, members):
    sizes = [1, 2, 17, 33, 64, 65, 100, 150, 160, 200, 232]  # 1,024 atoms
    mols = [w.single_molecule(n, seed=500 + n, n_species=S) for n in sizes + [1]]
    at = w.aev_table(S)
    pot = Potential.ensemble_from_tables(at, [w.mlp_table(S, seed=50 + k) for k in range(members)],
                                         precision="fp32", max_neighbors=128, deterministic=True)
    out = []
    for k in (len(sizes), len(sizes) + 1):
        s = w.pack_molecules(mols[:k], S)
        print(f"\n[case] S={S} members={members} N={s.n_atoms}", flush=True)
        out.append(pot.energy_forces(*to_dev(s)))
        pot.check()
    (E0, F0), (E1, F1) = out
    assert F0.shape[0] == 1024 and F1.shape[0] == 1025
    assert torch.equal(E0, E1[:-1])
    assert torch.equal(F0, F1[:-1])
