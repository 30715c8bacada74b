"""The rows' order in the fused network's tiles.

Large calls sort the rows of an element by their k-steps within windows of
1,024 rows.  A row's result does not depend on its tile, so in the
deterministic mode the energies and forces are the bits of calls small enough
to take the rows as they lie, and the weight gradients are the sum of theirs up
to the order of FP32 sums (1e-5).  Conformers of one molecule give many equal
masks and windows of a full and of a remaining part; eight elements give masks
of more than 32 bits; eight BF16 members take the adjoint of the ensemble.
"""
import numpy as np
import pytest
import torch

import workloads as w
from gpu_util import rel_rms, to_dev
from paper_2310_03121_amd import Potential

pytestmark = pytest.mark.gpu

CASES = {
    "fp32 7el": ("fp32", 7, 1, 96, 32),
    "fp32 8el": ("fp32", 8, 1, 96, 32),
    "fp32 4el": ("fp32", 4, 1, 270, 135),
    "bf16 7el 8 members": ("bf16", 7, 8, 70, 35),
}


@pytest.mark.parametrize("name", list(CASES))
def test_ordered_rows_agree_with_small_calls(name):
    prec, S, members, mols, part = CASES[name]
    extra = [w.single_molecule(n, seed=70 + n, n_species=S) for n in (1, 2, 33, 63)]
    base = w.conformer_batch(mols - len(extra), 64, seed=3, n_species=S)
    sys_ = w.pack_molecules([base.molecule(k) for k in range(mols - len(extra))] + extra, S)
    print(f"\n[case] {name} N={sys_.n_atoms}", flush=True)
    at = w.aev_table(S)
    mts = [w.mlp_table(S, seed=50 + k) for k in range(members)]
    pot = Potential.ensemble_from_tables(at, mts, precision=prec, max_neighbors=64,
                                         deterministic=True)
    pos, sp, off = to_dev(sys_)
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    up = torch.from_numpy(np.random.default_rng(6).normal(size=mols)).cuda()
    gw = None
    if members == 1:
        _, gw, _ = pot.backward(pos, sp, off, up)
        pot.check()
    ref = 0.0
    for m in range(0, mols, part):
        one = w.pack_molecules([sys_.molecule(k) for k in range(m, min(m + part, mols))], S)
        a, b = int(sys_.mol_offsets[m]), int(sys_.mol_offsets[min(m + part, mols)])
        p1, s1, o1 = to_dev(one)
        E1, F1 = pot.energy_forces(p1, s1, o1)
        pot.check()
        assert torch.equal(E1, E[m:m + part])
        assert torch.equal(F1, F[a:b])
        if gw is not None:
            _, g1, _ = pot.backward(p1, s1, o1, up[m:m + part].contiguous())
            pot.check()
            ref = ref + g1.double()
    if gw is not None:
        assert rel_rms(gw.cpu().numpy(), ref.cpu().numpy()) <= 1e-5
