"""Weights from vectors of any place and float type, and of too few entries.

A kernel reads the vector that the library is given, so one in host memory is
copied to the GPU first and one that is too short is refused before any launch.
"""
import numpy as np
import pytest
import torch

import workloads as w
from gpu_util import potential, to_dev
from paper_2310_03121_amd import Potential


def test_short_vector_is_refused():
    pot = object.__new__(Potential)  # no GPU: the check comes before the library
    pot.n_params = 10
    with pytest.raises(ValueError):
        pot.set_params(torch.zeros(9))


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_host_vectors(prec):
    print(f"\n[case] weights from host memory, {prec}", flush=True)
    s = w.single_molecule(24, seed=0)
    pot, _, _ = potential(4, prec)
    new = w.mlp_table(4, seed=9).flat()
    pos, sp, off = to_dev(s)
    E0, _ = pot.energy_forces(pos, sp, off)
    pot.set_params(torch.from_numpy(new).cuda())
    E1, F1 = pot.energy_forces(pos, sp, off)
    assert not torch.equal(E0, E1)
    long = torch.from_numpy(np.concatenate([new, new[:5]]))
    for host in (torch.from_numpy(new), torch.from_numpy(new).double(), long.pin_memory(),
                 torch.from_numpy(np.repeat(new, 2))[::2]):
        pot.set_params(torch.zeros(pot.n_params, device="cuda"))
        pot.set_params(host)
        E2, _ = pot.energy_forces(pos, sp, off)
        pot.check()
        assert torch.equal(E1, E2)
