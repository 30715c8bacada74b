"""The cell list's launches: the species sort beside the binning, and filling
from the places that the binning hands out (boxes of up to 8,192 cells), or the
scan in the binning's last workgroup (more cells).

The pair sets are those of the float32 predicate exactly, and the forces hold
the bars of the parity tests, for a single atom, workgroups that end on, before
and after an edge of 256 atoms, cells of many atoms, 8,000 and 9,261 cells that
are mostly empty, and a call on a workspace that a larger system has used.
"""
import numpy as np
import pytest
import torch

import oracle as o
import workloads as w
from gpu_util import check_forces, pair_set_from_ell, potential, to_dev
from oracle.neighbors import pair_list

pytestmark = pytest.mark.gpu

CASES = {
    "1 atom": (1, 20.8),
    "255 atoms": (255, 20.8),
    "256 atoms": (256, 20.8),
    "257 atoms": (257, 20.8),
    "900 atoms": (900, 20.8),
    "8,000 cells": (600, 20),
    "9,261 cells": (600, 21),
}


@pytest.mark.parametrize("name", list(CASES))
def test_box_pairs_and_forces(name):
    n, L = CASES[name]
    big = w.water_box(300, 20.8, seed=5)
    keep = np.random.default_rng(3).permutation(900)[:n]
    pot, at, mt = potential(4, "fp32")
    if isinstance(L, int):  # cells per side
        L *= at.rc_rad + 0.01
    pos, sp, off = to_dev(big)
    pot.energy_forces(pos, sp, off, big.box)
    pot.check()
    # some of the box's atoms, in a random order, in a box of another size:
    # clusters of up to 20.8 A in empty space
    p = np.ascontiguousarray(big.pos[keep], np.float32)
    if L > 30:
        p[: n // 2] += np.float32(L - 30.0)
    species = np.ascontiguousarray(big.species[keep])
    box = np.full(3, L, np.float32)
    moff = np.array([0, n], np.int32)
    print(f"\n[case] {name} N={n} L={L}", flush=True)
    pos, sp, off = (torch.from_numpy(x).cuda() for x in (p, species, moff))
    E, F = pot.energy_forces(pos, sp, off, box)
    pot.check()
    counts, nbr = pot.debug_neighbors(n)
    I, J = pair_set_from_ell(counts, nbr)
    Io, Jo = pair_list(p, moff, box, at.rc_rad)
    assert np.array_equal(I, Io) and np.array_equal(J, Jo)
    r = o.energy_forces(p, species, moff, box, aev_table=at, mlp_table=mt)
    scale = max(np.abs(r.E_atom).sum(), 1e-30)
    assert np.abs(E.cpu().numpy() - r.E).max() <= 1e-5 * scale
    check_forces(F.cpu().numpy(), r.F, "fp32", name)
