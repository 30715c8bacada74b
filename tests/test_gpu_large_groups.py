"""More rows of one element than a 32-bit range of bytes holds.

The networks' products read a tile's rows through ranges whose byte counts are
32 bits: an element's rows from a tile to the group's end can be more than
that (eight members' deltas of 256 columns are 8 KB a row in FP32).  The
molecules repeat one of 256, and in the deterministic mode a molecule's forces
are the same bits wherever it lies, so the large call has to repeat those of a
call of 1,024 atoms, its first and last tiles included.  The row counts put
the bytes of the first tile's range just past 2^32, and for three members (a
row of 7.5 chunks, whose last one loads past the range) past 2^31.
"""
import pytest
import torch

import workloads as w
from paper_2310_03121_amd import Potential

pytestmark = pytest.mark.gpu

CASES = {
    "fp32, 8 members of 256": ("fp32", 7, None, 8, 524_328),
    "bf16, 8 members of 256": ("bf16", 7, None, 8, 1_048_616),
    "fp32, 3 members of 160": ("fp32", 4, None, 3, 1_118_600),
    "bf16 layers, 8 members of 256": ("bf16", 4, (384, 256, 128, 96, 1), 8, 1_048_616),
}


@pytest.mark.parametrize("name", list(CASES))
def test_forces_repeat(name):
    prec, S, widths, members, n = CASES[name]
    print(f"\n[case] {name} N={n}", flush=True)
    at = w.aev_table(S)
    pot = Potential.ensemble_from_tables(
        at, [w.mlp_table(S, seed=50 + k, widths=widths) for k in range(members)], precision=prec,
        max_neighbors=16, deterministic=True)
    # molecules of four atoms of one element, 1 to 2 A apart
    corners = torch.tensor([[0, 0, 0], [1.2, 1.2, 0], [1.2, 0, 1.2], [0, 1.2, 1.2]])
    gen = torch.Generator().manual_seed(7)
    base = corners + 0.15 * torch.rand((256, 4, 3), generator=gen)

    def call(k):  # k molecules
        pos = base.reshape(-1, 3).repeat((k + 255) // 256, 1)[:4 * k].cuda()
        sp = torch.ones(4 * k, dtype=torch.int32, device="cuda")
        off = torch.arange(0, 4 * k + 1, 4, dtype=torch.int32, device="cuda")
        E, F = pot.energy_forces(pos, sp, off)
        pot.check()
        return E, F

    E0, F0 = call(256)
    assert bool(torch.isfinite(F0).all()) and float(F0.abs().max()) > 0.01
    E1, F1 = call(n // 4)
    reps = (n // 4 + 255) // 256
    assert torch.equal(E1, E0.repeat(reps)[:n // 4])
    bad = (F1 != F0.repeat(reps, 1)[:n]).any(1).nonzero().flatten()
    assert bad.numel() == 0, (bad.numel(), bad[:8].tolist())
