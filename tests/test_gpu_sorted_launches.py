"""Large calls that only the largest sizes reach.

One BF16 network above 32,768 rows takes its rows sorted by k-steps, in the
evaluation and in training (whose weight gradients then run in chunks of 1,024
rows); above 131,072 atoms the species sort and the pair scan take launches of
their own, with and without a box.  In the deterministic mode the energies and
forces of a batch are the bits of the same molecules in calls small enough to
take the other way, and the weight gradients the sum of theirs up to the order
of FP32 sums (1e-5).  Some molecules, and some atoms of the boxes (their
neighborhoods give their force exactly), are compared with the oracle.
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import potential, rel_rms, to_dev
from neighborhood import neighborhood_reference
from oracle.neighbors import pair_list

pytestmark = pytest.mark.gpu


def parts(s, pot, step, up=None):
    """(molecules, E, F, weight gradients) of `step` molecules at a time."""
    for m in range(0, s.n_mol, step):
        e = min(m + step, s.n_mol)
        one = w.pack_molecules([s.molecule(k) for k in range(m, e)], s.n_species)
        p1, s1, o1 = to_dev(one)
        E, F = pot.energy_forces(p1, s1, o1)
        pot.check()
        gw = None
        if up is not None:
            _, gw, _ = pot.backward(p1, s1, o1, up[m:e].contiguous())
            pot.check()
        yield (m, e), E, F, gw


@pytest.mark.parametrize("prec,mols,part", [("bf16", 530, 265), ("fp32", 400, 50)])
def test_training_on_many_rows(prec, mols, part):
    # 33,920 rows (sorted; halves of 16,960 are not); 25,600 rows in FP32,
    # where parts of 3,200 are not
    s = w.conformer_batch(mols, 64, seed=3)
    print(f"\n[case] training {prec} N={s.n_atoms}", flush=True)
    pot, _, _ = potential(7, prec, max_neighbors=64, deterministic=True)
    pos, sp, off = to_dev(s)
    up = torch.from_numpy(np.random.default_rng(6).normal(size=mols)).cuda()
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    gp, gw, E2 = pot.backward(pos, sp, off, up)
    pot.check()
    assert torch.equal(E, E2)
    ref = 0.0
    for (m, e), E1, F1, g1 in parts(s, pot, part, up):
        a, b = int(s.mol_offsets[m]), int(s.mol_offsets[e])
        assert torch.equal(E1, E[m:e])
        assert torch.equal(F1, F[a:b])
        ref = ref + g1.double()
    err = rel_rms(gw.cpu().numpy(), ref.cpu().numpy())
    print(f"weight gradients {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_batch_beyond_the_fused_sort(prec):
    mols = 2060  # 131,840 atoms; BF16 rows of 412 molecules are not sorted
    s = w.conformer_batch(mols, 64, seed=1)
    print(f"\n[case] batch {prec} N={s.n_atoms}", flush=True)
    pot, at, mt = potential(7, prec, max_neighbors=64, deterministic=True)
    pos, sp, off = to_dev(s)
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    counts, nbr = pot.debug_neighbors(s.n_atoms)
    for m in (0, 1029, 2059):
        a, b = int(s.mol_offsets[m]), int(s.mol_offsets[m + 1])
        one = s.molecule(m)
        r = o.energy_forces(one, aev_table=at, mlp_table=mt)
        tol = 1e-5 if prec == "fp32" else 1e-2
        assert abs(float(E[m]) - r.E[0]) <= tol * np.abs(r.E_atom).sum()
        assert rel_rms(F[a:b].cpu().numpy(), r.F) <= tol
        I, J = pair_list(one.pos, one.mol_offsets, None, at.rc_rad)
        for i in range(64):
            got = nbr[a + i, :int(counts[a + i, 0])].cpu().numpy() - a
            assert np.array_equal(np.sort(got), J[I == i])
    for (m, e), E1, F1, _ in parts(s, pot, 412):
        assert torch.equal(E1, E[m:e])
        assert torch.equal(F1, F[64 * m:64 * e])


@pytest.mark.parametrize("reps", [(1, 1, 30), (3, 3, 4)], ids=["4,608 cells", "10,800 cells"])
def test_box_beyond_the_fused_sort(reps):
    """Boxes of 4,500 atoms of water side by side: 135,000 and 162,000 atoms,
    in cells that the filling scans itself, and in more than it can."""
    cell = w.water_box(1500, 35.5, seed=2, n_species=4)
    L = 35.5
    shift = np.array([[i, j, k] for i in range(reps[0]) for j in range(reps[1])
                      for k in range(reps[2])], np.float64) * L
    pos = (cell.pos.astype(np.float64)[None] + shift[:, None]).reshape(-1, 3).astype(np.float32)
    n = pos.shape[0]
    s = w.System(pos, np.tile(cell.species, len(shift)), np.array([0, n], np.int32),
                 (np.array(reps) * L).astype(np.float32), 4, "waters")
    print(f"\n[case] box {reps} N={n}", flush=True)
    assert n > 131072
    pot, at, mt = potential(4, "fp32", max_neighbors=128)
    p, sp, off = to_dev(s)
    E, F = pot.energy_forces(p, sp, off, s.box)
    pot.check()
    counts, nbr = pot.debug_neighbors(n)
    F = F.cpu().numpy()
    ks = np.random.default_rng(5).choice(n, 16, replace=False)
    ref = []
    for k in ks:
        f, near = neighborhood_reference(s, at, mt, int(k))
        ref.append(f)
        assert set(nbr[k, :int(counts[k, 0])].tolist()) == near
    err = rel_rms(F[ks], np.array(ref))
    print(f"forces on {len(ks)} atoms {err:.2e}", flush=True)
    assert err <= 1e-5
