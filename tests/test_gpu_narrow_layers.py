"""dE/dG of BF16 layer kernels whose K is shorter than the weight ring.

A first hidden layer of 32, 64 or 96 columns gives products of one to three
k-steps in a ring of four, over several passes of columns.  The ring has to
stay inside the weights: behind the last element's lie the biases, which here
are numbers whose low halves are NaN as bfloat16.  All atoms are of the last
element.  Bars: those of the BF16 path.
"""
import numpy as np
import pytest

import oracle as o
import workloads as w
from gpu_util import check_forces, to_dev
from paper_2310_03121_amd import Potential

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [1, 2, 3])
@pytest.mark.parametrize("w1", [32, 64, 96])
def test_forces(w1, members):
    s = w.single_molecule(48, seed=5, n_species=4)
    s.species[:] = 3
    print(f"\n[case] widths 384-{w1}-64-32, {members} members", flush=True)
    at = w.aev_table(4)
    mts = [w.mlp_table(4, seed=30 + k, widths=(384, w1, 64, 32, 1)) for k in range(members)]
    for mt in mts:
        for b in mt.b:
            for x in b:
                x.view(np.uint32)[:] = (x.view(np.uint32) & 0xffff0000) | 0x7fc0
    pot = Potential.ensemble_from_tables(at, mts, precision="bf16")
    pos, sp, off = to_dev(s)
    _, F = pot.energy_forces(pos, sp, off)
    pot.check()
    r = o.ensemble_energy_forces(s, aev_table=at, mlp_tables=mts)
    check_forces(F.cpu().numpy(), r.F, "bf16", f"w1={w1}")
