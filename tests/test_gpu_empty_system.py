"""A system of no atoms, with and without a box.

Nothing is staged, sorted or searched, but the kernels that follow read the
group table, so it has to say so whatever the workspace held: the calls run on
a workspace whose every byte is set.  The energy is zero, the status clean.
"""
import numpy as np
import pytest
import torch

from gpu_util import potential

pytestmark = pytest.mark.gpu

BOXES = {"no box": (None, False), "box": (np.full(3, 20.8, np.float32), False),
         "box of 9,261 cells": (np.full(3, 21 * 5.11, np.float32), False),
         "triclinic": (np.array([[21, 0, 0], [3, 21, 0], [-2, 4, 21]], np.float32), True)}


def empty_call(prec, box):
    box, tric = BOXES[box]
    pot, _, _ = potential(7, prec, triclinic=tric)
    pos = torch.empty((0, 3), dtype=torch.float32, device="cuda")
    sp = torch.empty(0, dtype=torch.int32, device="cuda")
    off = torch.zeros(2, dtype=torch.int32, device="cuda")
    pot.workspace(0, 1, box).fill_(0x5a)
    return pot, pos, sp, off, box


@pytest.mark.parametrize("box", list(BOXES))
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_energy_and_forces(prec, box):
    print(f"\n[case] no atoms, {prec}, {box}", flush=True)
    pot, pos, sp, off, b = empty_call(prec, box)
    E, F = pot.energy_forces(pos, sp, off, b, forces=False)
    pot.check()
    assert E.tolist() == [0.0]
    E = torch.full((1,), 3.0, dtype=torch.float64, device="cuda")
    F = torch.full((1, 3), 2.0, dtype=torch.float32, device="cuda")
    pot.workspace(0, 1, b).fill_(0x5a)
    pot.energy_forces(pos, sp, off, b, out=(E, F))
    pot.check()
    assert E.tolist() == [0.0] and bool((F == 2.0).all())


@pytest.mark.parametrize("box", ["no box", "box"])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_weight_gradients(prec, box):
    print(f"\n[case] weight gradients of no atoms, {prec}, {box}", flush=True)
    pot, pos, sp, off, b = empty_call(prec, box)
    up = torch.full((1,), 2.0, dtype=torch.float64, device="cuda")
    _, gw, E = pot.backward(pos, sp, off, up, b)
    pot.check()
    assert E.tolist() == [0.0]
    assert gw.numel() == pot.n_params and bool((gw == 0.0).all())
