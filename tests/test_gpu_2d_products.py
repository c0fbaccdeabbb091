"""The matrix-vector products of 2D plans (csrc/gemv.hip and the N_z = 1 step kernels) against the oracle: row
blocks of 16 (pairs of 32) with remainders, contractions shorter and longer than the 32 groups, odd
N_r (a middle node), a radial chop, orders without degrees.

Tolerance: the parity bar of the FP64 paths (1e-12 normwise).
"""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle import timestep as ts
from oracle.grid import Grid
from oracle.rhs import rhs_scalar
from oracle.transform import Tables, backward, forward

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-12


@pytest.mark.parametrize("case", [
    # nr, nphi, nrc
    (2, 4, 0), (3, 4, 0), (16, 8, 0), (17, 6, 0), (31, 12, 0), (32, 12, 0), (33, 16, 9), (64, 10, 63), (97, 8, 0),
    (130, 6, 0), (257, 4, 0),
])
def test_products(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import MLG_RHS_KPP, Plan
    nr, nphi, nrc = case
    print("2D products", case, flush=True)
    g = Grid(nr, nphi, 1, 1.2, nrc=nrc)
    t = Tables(g)
    plan = Plan(nr, nphi, 1, 1.2, nrc=nrc)
    phys = np.random.default_rng(nr).standard_normal((1, nr, nphi))
    spec, back = plan.empty_spec(), plan.empty_phys()
    plan.forward(torch.from_numpy(phys).cuda(), spec)
    ref = forward(phys, g, t)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < TOL
    plan.backward(spec, back)
    assert rel(back.cpu().numpy(), backward(ref, g, t)) < TOL
    S = [synth.geometric_spectrum(g.M, g.nrc, 1, g.nzc, seed=i, a=0.8, b=0.8, c=1.0) for i in (1, 2, 3)]
    s, a1, a0 = (torch.from_numpy(to_lib(X)).cuda() for X in S)
    out = torch.full_like(s, float("nan"))       # every entry is written, the masked orders as zero
    plan.rhs_scalar(MLG_RHS_KPP, 0.25, s, out)
    got, ref = from_lib(out.cpu().numpy(), g.M, g.nrc), rhs_scalar(S[0], g, t, "kpp", 0.25)
    assert rel(got, ref) < TOL and np.all(got[g.dealias_m() + 1:] == 0)
    nu, nu_h, p, dt = 0.02, 1e-5, 4, 0.02
    diss = ts.Dissipation(g, nu, nu_h, p)
    plan.step_setup(nu, nu_h, p, dt)
    plan.step_abcn(s, a1, a0, out)
    assert rel(from_lib(out.cpu().numpy(), g.M, g.nrc), ts.abcn_step(S[0], S[1], S[2], dt, diss)) < TOL
    plan.step_febe(0, s, a1, out)
    assert rel(from_lib(out.cpu().numpy(), g.M, g.nrc), diss.apply_inverse(S[0] + dt * S[1], dt)) < TOL
