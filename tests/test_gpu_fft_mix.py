"""The two-pass transforms of every length n = R1 R2 they serve (csrc/fft_mix.hip) against the oracle, on few
lines: ragged last blocks, an order stored at the Nyquist index, dealiasing on and off.

Tolerance: the parity bar of the FP64 paths (1e-12 normwise); a transform's own rounding is below
log2(n) eps, 2e-15.
"""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import VecTables, rhs_scalar, rhs_tp
from oracle.transform import Tables, backward, forward

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-12
PAIRS = [4, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81, 90,
         96, 100, 108, 120, 128, 135, 144, 150, 160]
WIDE = [180, 192, 225, 240]


def _plan(*a, **k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    return Plan(*a, **k)


@pytest.mark.parametrize("n", PAIRS + WIDE)
def test_z_transform(n):
    nr, nphi = 5, 4
    print("z transform", n, flush=True)
    g = Grid(nr, nphi, n, 0.9, lz=2.0)
    t = Tables(g)
    plan = _plan(nr, nphi, n, 0.9, 2.0)
    s = np.random.default_rng(n).standard_normal((n, nr, nphi))
    spec, back = plan.empty_spec(), plan.empty_phys()
    plan.forward(torch.from_numpy(s).cuda(), spec)
    ref = forward(s, g, t)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < TOL
    plan.backward(spec, back)
    assert rel(back.cpu().numpy(), backward(ref, g, t)) < TOL


@pytest.mark.parametrize("nr, nz", [(5, 1), (7, 3), (40, 9)])
@pytest.mark.parametrize("n", PAIRS + WIDE)
def test_phi_scalar_stages(n, nr, nz):
    """Transform pair with the Nyquist order stored, then both scalar terms (in place, masked) on an odd number of lines."""
    M = n // 2 + 1
    print("phi scalar stages", n, nr, nz, flush=True)
    from paper_2609_18026_amd import MLG_RHS_KPP, MLG_RHS_U2
    g = Grid(nr, n, nz, 0.9, lz=2.0, nphic=M)
    t = Tables(g)
    plan = _plan(nr, n, nz, 0.9, 2.0, nphic=M)
    s = np.random.default_rng(n).standard_normal((nz, nr, n))
    spec, back = torch.full_like(plan.empty_spec(), float("nan")), plan.empty_phys()
    plan.forward(torch.from_numpy(s).cuda(), spec)
    ref = forward(s, g, t)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < TOL
    plan.backward(spec, back)
    assert rel(back.cpu().numpy(), backward(ref, g, t)) < TOL
    S = synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=4, a=0.8, b=0.8, c=0.8)
    for kind, name in ((MLG_RHS_U2, "u2"), (MLG_RHS_KPP, "kpp")):
        out = torch.full_like(spec, float("nan"))
        plan.rhs_scalar(kind, 0.25, torch.from_numpy(to_lib(S)).cuda(), out)
        got = from_lib(out.cpu().numpy(), g.M, g.nrc)
        assert rel(got, rhs_scalar(S, g, t, name, 0.25)) < TOL and np.all(got[g.dealias_m() + 1:] == 0)


@pytest.mark.parametrize("dealias", [0, 1])
@pytest.mark.parametrize("n", PAIRS)
def test_phi_vector_stage(n, dealias):
    nr, nz = 7 + n % 2, 3      # 21 or 24 lines: partial blocks of 8, 16 and 32 lines
    M = n // 2 + 1 - dealias   # without dealiasing also the order n // 2
    U = (0.3, -0.2, 0.5)
    print("phi vector stage", n, dealias, flush=True)
    g = Grid(nr, n, nz, 0.8, lz=3.0, nphic=M)
    psi = synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=2)
    chi = synth.geometric_spectrum(g.M, g.nrc, nz, g.nzc, seed=3)
    taps = {}
    rhs_tp(psi, chi, g, VecTables(g), U=U, dealias=bool(dealias), taps=taps)
    plan = _plan(nr, n, nz, 0.8, 3.0, nphic=M, dealias=dealias)
    tp = plan.taps_buffer()
    args = [torch.from_numpy(to_lib(psi)).cuda(), torch.from_numpy(to_lib(chi)).cuda()]
    po, co, pn, cn = (plan.empty_spec() for _ in range(4))
    plan.rhs_tp(*args, po, co, U=U, taps=tp)
    plan.rhs_tp(*args, pn, cn, U=U)          # the instance without the tap stores
    pe = plan.layout.phys_elems
    got = tp.cpu().numpy()
    nodal = got[:9 * pe].reshape(9, nz, nr, n)
    for i, ref in enumerate(list(taps["u"]) + list(taps["w"]) + list(taps["N"])):
        assert rel(nodal[i], ref) < TOL, (i, rel(nodal[i], ref))
    src = got[9 * pe:].view(np.complex128).reshape(3, plan.tau, nz)
    scale = max(np.linalg.norm(taps[k]) for k in "CKZ")
    for i, k in enumerate("CKZ"):
        assert np.linalg.norm(from_lib(src[i], g.M, g.nrc) - taps[k]) < TOL * scale, k
    assert rel(pn.cpu().numpy(), po.cpu().numpy()) < 1e-11 and rel(cn.cpu().numpy(), co.cpu().numpy()) < 1e-11
