"""Partial sums of the axial modal energy where their split can go wrong: one, five, 36 and 270 axial slots (a slot count
that is no power of two, one past the block), fewer rows than row groups, thousands of rows.  Sums of squares, 1e-12 normwise."""
import numpy as np
import pytest

import synth
from helpers import rel, to_lib
from oracle.diagnostics import axial_modal_energy
from oracle.grid import Grid
from oracle.rhs import VecTables

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nr, nphi, nz", [(2, 2, 1), (3, 2, 5), (96, 64, 1), (17, 6, 36), (150, 40, 12), (6, 4, 270)])
def test_energy_parts(nr, nphi, nz):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    print("energy parts", nr, nphi, nz, flush=True)
    g = Grid(nr, nphi, nz, 0.9, lz=3.0)
    psi = synth.geometric_spectrum(g.M, g.nrc, g.nz, g.nzc, seed=21, a=0.85, b=0.8, c=0.8)
    chi = synth.geometric_spectrum(g.M, g.nrc, g.nz, g.nzc, seed=22, a=0.85, b=0.8, c=0.8)
    want = axial_modal_energy(psi, chi, g, VecTables(g))
    plan = Plan(nr, nphi, nz, 0.9, 3.0, dealias=1)
    got = plan.energy(torch.from_numpy(to_lib(psi)).cuda(), torch.from_numpy(to_lib(chi)).cuda()).cpu().numpy()
    assert rel(got, want) < 1e-12, rel(got, want)
