"""The adjoint's paths: long lists and crowded neighborhoods.

Molecules of up to 10,000 atoms, larger batches (workgroups with a window of
atoms) and boxes take three kernels.  Each has limits beyond which it goes
another way: 16 angular neighbors of an atom (short lists), 64 entries (one
per lane), 192 pairs of angular neighbors (the LDS table), 64 angular
neighbors (the LDS entries), three elements among them (the staged dE/dG
blocks).  Clusters of rising density lie on both sides of each.  In a large
batch they stand between many small molecules and are compared alone.

Bar: the FP32 force bar (1e-5 relative, held with about 150 pairs per atom)
grows with the square root of the pairs an atom sums, to 5e-5 for the densest
(about 2,900 pairs).
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import potential, rel_rms, to_dev

pytestmark = pytest.mark.gpu


def cluster(n, side, seed, S):
    rng = np.random.default_rng(seed)
    pos = w.random_molecule(n, side, 0.9, rng).astype(np.float32)
    sp = rng.integers(0, S, n).astype(np.int32)
    return w.System(pos, sp, np.array([0, n], np.int32), None, 7, f"cluster{n}")


def clusters():
    # most angular neighbors of an atom: 13, 26, 47, 77, 38
    return [cluster(30, 7.0, 1, 7), cluster(60, 7.5, 2, 3), cluster(70, 6.2, 3, 4),
            cluster(110, 6.0, 4, 2), cluster(150, 9.0, 5, 7)]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("fill", [0, 400])
def test_crowded_molecules(fill, prec):
    dense = clusters()
    small = [w.single_molecule(10 + k % 40, seed=3000 + k, n_species=7) for k in range(fill)]
    mols = dense[:2] + small + dense[2:]
    s = w.pack_molecules(mols, 7)
    print(f"\n[case] crowded molecules {prec} N={s.n_atoms}", flush=True)
    assert (s.n_atoms > 10000) == (fill > 0)
    pot, at, mt = potential(7, prec, max_neighbors=192)
    pos, sp, off = to_dev(s)
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    counts, _ = pot.debug_neighbors(s.n_atoms)
    na = counts[:, 1]
    assert int(na.max()) > 64 and bool(((na > 16) & (na <= 64)).any())
    F = F.cpu().numpy()
    for m in [0, 1] + list(range(2 + fill, s.n_mol)):
        a, b = s.mol_offsets[m], s.mol_offsets[m + 1]
        r = o.energy_forces(mols[m], aev_table=at, mlp_table=mt)
        err = rel_rms(F[a:b], r.F)
        print(f"molecule {m} ({b - a} atoms): {err:.2e}", flush=True)
        assert err <= (5e-5 if prec == "fp32" else 1e-2)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("atoms,S", [(90, 2), (330, 7)])
def test_crowded_box(atoms, S, prec):
    # boxes of 10.4 A: up to 21 and 75 angular neighbors, two and seven elements
    rng = np.random.default_rng(atoms)
    pos = w.random_molecule(atoms, 9.5, 0.9, rng).astype(np.float32)
    s = w.System(pos, rng.integers(0, S, atoms).astype(np.int32),
                 np.array([0, atoms], np.int32), np.full(3, 10.4, np.float32), 7, "crowded")
    print(f"\n[case] crowded box {prec} N={atoms}", flush=True)
    pot, at, mt = potential(7, prec, max_neighbors=256)
    p, sp, off = to_dev(s)
    E, F = pot.energy_forces(p, sp, off, s.box)
    pot.check()
    r = o.energy_forces(s, aev_table=at, mlp_table=mt)
    err = rel_rms(F.cpu().numpy(), r.F)
    print(f"{err:.2e}", flush=True)
    assert err <= (5e-5 if prec == "fp32" else 1e-2)
