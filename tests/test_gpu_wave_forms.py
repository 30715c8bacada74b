"""Calls on both sides of the rules that choose how many atoms a wave takes.

Above 16,384 atoms the pair scan (molecules of at most 512 atoms in the mean)
and the symmetry functions (of at most 160) give each wave four atoms instead
of one.  The pair sets are those of the float32 predicate exactly on either
side; the symmetry functions' four-atom waves, with lists that fit their 64
entries and pairs that fit the shared table, with more pairs, and with longer
lists, give the features of the deterministic mode (one atom per wave) bit for
bit, and so its energies.  Forces are its up to the order of FP32 sums of a few
hundred terms (5e-6), and some molecules' are the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import pair_set_from_ell, potential, rel_rms, to_dev
from oracle.neighbors import pair_list

pytestmark = pytest.mark.gpu


def copies(base, sizes, seed, S, jitter=0.05):
    """Molecules of the first `sizes` atoms of one molecule, jittered."""
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    pos = np.concatenate([base.pos[:k] for k in sizes]).astype(np.float64)
    pos += rng.normal(0.0, jitter, pos.shape)
    sp = np.concatenate([base.species[:k] for k in sizes]).astype(np.int32)
    return w.System(pos.astype(np.float32), sp, off, None, S, "copies")


@pytest.mark.parametrize("sizes", [[512] * 32, [529] * 31, [3000] + [610] * 22, [16500]],
                         ids=["32x512", "31x529", "3000+22x610", "16500"])
def test_pairs_around_the_mean_size(sizes):
    base = w.single_molecule(max(sizes[0], 610), seed=8, n_species=4)
    if sizes == [16500]:  # one molecule: copies of a small one side by side
        small = w.single_molecule(500, seed=8, n_species=4)
        pos = np.concatenate([small.pos + np.float32([24.0 * k, 0, 0]) for k in range(33)])
        base = w.System(pos, np.tile(small.species, 33), np.array([0, 16500], np.int32), None, 4,
                        "row")
    s = copies(base, sizes, 3, 4)
    print(f"\n[case] molecules of {sizes[0]}, N={s.n_atoms}", flush=True)
    assert s.n_atoms >= 16384
    pot, at, _ = potential(4, "fp32", max_neighbors=64)
    pos, sp, off = to_dev(s)
    pot.energy_forces(pos, sp, off)
    pot.check()
    counts, nbr = pot.debug_neighbors(s.n_atoms)
    I, J = pair_set_from_ell(counts, nbr)
    Io, Jo = pair_list(s.pos, s.mol_offsets, None, at.rc_rad)
    assert np.array_equal(I, Io) and np.array_equal(J, Jo)


def molecule(n, seed, S, density):
    """n atoms, density times 24 of them in (10 A)^3."""
    rng = np.random.default_rng(seed)
    pos = w.random_molecule(n, 10.0 * (n / (24.0 * density)) ** (1 / 3), 0.9, rng)
    return w.System(pos.astype(np.float32), rng.integers(0, S, n).astype(np.int32),
                    np.array([0, n], np.int32), None, S, f"mol{n}")


def four_atom_waves(counts):
    """(fit with one table, fit with their own tables, do not fit) over the
    groups of four consecutive atoms."""
    c = counts.cpu().numpy().astype(np.int64)
    c = c[:len(c) // 4 * 4].reshape(-1, 4, 2)
    entries = ((c[..., 0] + 3) // 4 * 4).sum(1)
    pairs = ((c[..., 1] * (c[..., 1] - 1) // 2 + 3) // 4 * 4).sum(1)
    fit = entries <= 64
    return int((fit & (pairs <= 64)).sum()), int((fit & (pairs > 64)).sum()), int((~fit).sum())


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("S", [4, 5, 7, 8])
def test_symmetry_functions_of_crowded_batches(S, prec):
    kinds = [molecule(64, 5, S, 1), molecule(64, 6, S, 3), molecule(13, 7, S, 3),
             molecule(33, 9, S, 1), molecule(150, 10, S, 3)]
    s = w.pack_molecules([kinds[(k * k + k // 3) % 5] for k in range(260)], S)
    rng = np.random.default_rng(4)
    s.pos += rng.normal(0.0, 0.05, s.pos.shape).astype(np.float32)
    print(f"\n[case] crowded batch S={S} {prec} N={s.n_atoms}", flush=True)
    assert 16384 < s.n_atoms < 160 * s.n_mol
    pot, at, mt = potential(S, prec, max_neighbors=128)
    pos, sp, off = to_dev(s)
    E, F = pot.energy_forces(pos, sp, off)
    pot.check()
    counts, _ = pot.debug_neighbors(s.n_atoms)
    waves = four_atom_waves(counts)
    print("waves of one table, own tables, long lists:", waves, flush=True)
    assert min(waves) > 20
    G = pot.debug_aev(pos, sp, off)
    pot.set_deterministic(True)
    G1 = pot.debug_aev(pos, sp, off)
    assert torch.equal(G, G1)
    E1, F1 = pot.energy_forces(pos, sp, off)
    pot.check()
    assert torch.equal(E, E1)
    err = rel_rms(F.cpu().numpy(), F1.cpu().numpy())
    print(f"forces against the deterministic mode: {err:.2e}", flush=True)
    assert err <= 5e-6
    for m in (0, 1, 2, 100):
        a, b = s.mol_offsets[m], s.mol_offsets[m + 1]
        r = o.energy_forces(s.molecule(m), aev_table=at, mlp_table=mt)
        err = rel_rms(F[a:b].cpu().numpy(), r.F)
        print(f"molecule {m} ({b - a} atoms): {err:.2e}", flush=True)
        assert err <= (5e-5 if prec == "fp32" else 1e-2)
