"""Calls on both sides of the rules that choose how many atoms a wave takes.

Above 16,384 atoms the pair scan (molecules of at most 512 atoms in the mean)
gives each wave four atoms instead of one.  The pair sets are those of the
float32 predicate exactly on either side.
"""
import numpy as np
import pytest

import workloads as w
from gpu_util import pair_set_from_ell, potential, to_dev
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
