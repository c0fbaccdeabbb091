"""Banded solves of the vector term at the run lengths' edges: columns of 32 n + 1 and 32 n + 2 degrees (the longest that n
rows a run hold, and one more).  With taps the runs have 8 or 16 rows, and that path is held against the oracle by its
backward error elsewhere; without taps the shortest run is taken, and the same operations in the same order leave the same bits."""
import numpy as np
import pytest

import synth
from helpers import to_lib
from oracle.grid import Grid

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nrc", [2, 33, 65, 66, 97, 98, 129, 130, 161, 162, 193, 194, 225, 226, 256, 258])
def test_solve_run_lengths(nrc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    nr, nphi, nz, U = nrc + nrc % 2, 8, 4, (0.1, 0.3, -0.2)
    print("solve runs", nrc, flush=True)
    g = Grid(nr, nphi, nz, 1.0, lz=3.0, nrc=nrc)
    psi, chi = (torch.from_numpy(to_lib(synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=q, a=0.9, b=0.85, c=0.85))).cuda()
                for q in (31, 32))
    plan = Plan(nr, nphi, nz, 1.0, 3.0, nrc=nrc, dealias=1)
    out = [plan.empty_spec() for _ in range(4)]
    for o in out:
        o.fill_(float("nan"))
    plan.rhs_tp(psi, chi, out[0], out[1], U=U)
    plan.rhs_tp(psi, chi, out[2], out[3], U=U, taps=plan.taps_buffer())
    torch.cuda.synchronize()
    for a, b in ((out[0], out[2]), (out[1], out[3])):
        assert torch.isfinite(torch.view_as_real(a)).all()
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
