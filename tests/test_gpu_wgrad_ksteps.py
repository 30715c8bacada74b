"""Layer 1's weight gradients over the feature rows' k-steps.

Each chunk of an element's rows lists, per k-step of 32 feature columns, the
rows that have it; rows are stored without their other k-steps.  The cases put
an element's row count below, at and past the smallest chunk (128 rows) and the
stage sizes (32 and 64 rows), with absent elements and absent k-steps, both
width sets and a system of several chunks per element; a larger call on the
same handle goes first, so that what lies between the stored k-steps is not
zero.  Bars per (element, layer) block: FP32 sums of at most a few thousand
terms, 1e-4; BF16 operands carry up to 2^-9 each, 3e-2.
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import potential, rel_rms, to_dev

pytestmark = pytest.mark.gpu

CASES = {
    "1 atom": (7, lambda: w.single_molecule(1, seed=3)),
    "2 atoms": (7, lambda: w.single_molecule(2, seed=3)),
    "65 atoms": (7, lambda: w.single_molecule(65, seed=5)),
    "128 x 2 rows": (7, lambda: w.conformer_batch(128, 2, seed=7)),
    "129 x 2 rows": (7, lambda: w.conformer_batch(129, 2, seed=7)),
    "5 x 60": (4, lambda: w.pack_molecules(
        [w.single_molecule(60, seed=k, n_species=4) for k in range(5)], 4)),
    "water 3,600": (4, lambda: w.water_box(1200, 33.1, seed=5)),
    "100 x 64": (7, lambda: w.conformer_batch(100, 64, seed=2)),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_weight_gradients_by_kstep(prec, name):
    S, make = CASES[name]
    s = make()
    print(f"\n[case] {prec} {name}: S={S} N={s.n_atoms}", flush=True)
    pot, at, mt = potential(S, prec)
    first = w.pack_molecules([w.single_molecule(64, seed=40 + k, n_species=S)
                              for k in range(s.n_atoms // 64 + 2)], S)
    pos, sp, off = to_dev(first)
    pot.backward(pos, sp, off, torch.ones(first.n_mol, dtype=torch.float64, device="cuda"))
    pot.check()
    pos, sp, off = to_dev(s)
    dLdE = np.random.default_rng(4).normal(size=s.n_mol)
    up = torch.from_numpy(dLdE).cuda()
    _, gw, _ = pot.backward(pos, sp, off, up, box=s.box)
    pot.check()
    _, gw2, _ = pot.backward(pos, sp, off, up, box=s.box)
    pot.check()
    ref, _ = o.weight_gradients(s, aev_table=at, mlp_table=mt, dL_dE=dLdE)
    gw, gw2 = gw.cpu().numpy(), gw2.cpu().numpy()
    bar = 1e-4 if prec == "fp32" else 3e-2
    k = 0
    present = set(int(x) for x in s.species)
    for e in range(S):
        for l in range(4):
            n = mt.W[e][l].size + mt.b[e][l].size
            blk = slice(k, k + n)
            if e in present:
                assert rel_rms(gw[blk], ref[blk]) <= bar, (e, l)
                assert rel_rms(gw2[blk], ref[blk]) <= bar, (e, l)
            else:
                assert np.all(gw[blk] == 0)
            k += n
