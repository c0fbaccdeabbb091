"""The curl source C of the projection products at the edges of their tiles (63 to 65, 100, 101 and 129 pairs of degrees), from the
library's own nodal N.  C = -Q (N_phi / r) - i m Pbar (N_r / r) cancels for flows whose N is nearly a gradient, so the bound
is the 1e-12 of the FP64 paths times the norms of its two terms."""
import numpy as np
import pytest

import synth
from helpers import from_lib, to_lib
from oracle.grid import Grid
from oracle.rhs import VecTables, _mixed_forward, dealias_mask, projection_sources

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nrc", [126, 127, 130, 200, 201, 258])
def test_curl_source(nrc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    nr, nphi, nz = nrc + nrc % 2, 12, 8
    print("curl source", nrc, flush=True)
    g = Grid(nr, nphi, nz, 1.0, lz=3.0, nrc=nrc)
    vt = VecTables(g)
    psi, chi = (synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=q, a=0.8, b=0.8, c=0.8) for q in (41, 42))
    plan = Plan(nr, nphi, nz, 1.0, 3.0, nrc=nrc, dealias=1)
    tp, po, co = plan.taps_buffer(), plan.empty_spec(), plan.empty_spec()
    plan.rhs_tp(torch.from_numpy(to_lib(psi)).cuda(), torch.from_numpy(to_lib(chi)).cuda(), po, co, U=(0.1, 0.3, -0.2), taps=tp)
    got, pe = tp.cpu().numpy(), plan.layout.phys_elems
    N = got[6 * pe:9 * pe].reshape(3, nz, nr, nphi)
    C = from_lib(got[9 * pe:].view(np.complex128).reshape(3, plan.tau, nz)[0], g.M, g.nrc)
    mask = dealias_mask(g)[:, None, :]
    want = projection_sources(N[0], N[1], N[2], g, vt)[0] * mask
    a, b = (_mixed_forward(f / g.r[None, :, None], g) for f in (N[0], N[1]))
    scale = sum(np.linalg.norm((np.stack([t[m] * g.w[None, :] @ f[m] * c(m) for m in range(g.M)]) * mask).ravel())
                for t, f, c in ((vt.Q, b, lambda m: 1.0), (vt.P, a, float)))
    err = np.linalg.norm((C - want).ravel())
    print("  error", err, "terms", scale, "C", np.linalg.norm(want.ravel()), flush=True)
    assert err < 1e-12 * scale
