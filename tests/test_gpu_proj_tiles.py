"""Sources of the vector term at the edges of the projection's tiles: 63 to 65 pairs of degrees (one and two row blocks of one
group a wavefront), 100 and 101 (one group and two), 129 (two row blocks of two groups); 1e-12 normwise against the oracle."""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import VecTables, rhs_tp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nrc", [126, 127, 130, 200, 201, 258])
def test_projection_tiles(nrc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    nr, nphi, nz, U = nrc + nrc % 2, 12, 8, (0.1, 0.3, -0.2)
    print("projection tiles", nrc, flush=True)
    g = Grid(nr, nphi, nz, 1.0, lz=3.0, nrc=nrc)
    psi, chi = (synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=q, a=0.8, b=0.8, c=0.8) for q in (41, 42))
    taps = {}
    rhs_tp(psi, chi, g, VecTables(g), U=U, dealias=True, taps=taps)
    plan = Plan(nr, nphi, nz, 1.0, 3.0, nrc=nrc, dealias=1)
    tp, po, co = plan.taps_buffer(), plan.empty_spec(), plan.empty_spec()
    plan.rhs_tp(torch.from_numpy(to_lib(psi)).cuda(), torch.from_numpy(to_lib(chi)).cuda(), po, co, U=U, taps=tp)
    torch.cuda.synchronize()
    src = tp.cpu().numpy()[9 * plan.layout.phys_elems:].view(np.complex128).reshape(3, plan.tau, nz)
    for i, nm in ((1, "K"), (2, "Z")):
        err = rel(from_lib(src[i], g.M, g.nrc), taps[nm])
        print("  rel", nm, err, flush=True)
        assert err < 1e-12, (nm, err)
