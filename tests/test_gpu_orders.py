"""Azimuthal stages with every kept order excited, at every length they serve (csrc/fft_mix.hip, csrc/batch.hip): N_r above the
number of orders, so that no order is empty, and flat spectra over the orders.  Bounds as for the other FP64 paths, 1e-12
normwise; every kept order of every compared quantity holds at least 1e-7 of its norm, so that a mistake in one order shows."""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import VecTables, rhs_scalar, rhs_tp
from oracle.transform import Tables, backward, forward

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL, SHARE = 1e-12, 1e-7
NZ = 5
PAIRS = [4, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81, 90,
         96, 100, 108, 120, 128, 135, 144, 150, 160]
WIDE = [180, 192, 225, 240]
SMOOTH = sorted({2 ** i * 3 ** j * 5 ** k for i in range(9) for j in range(6) for k in range(4)} - {1})
SMOOTH = [n for n in SMOOTH if n <= 256]


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_18026_amd as m
    return m


def _excited(S, orders):
    """S [m, ...]: the smallest share of an order in the norm."""
    norms = np.linalg.norm(S.reshape(S.shape[0], -1), axis=1)
    return norms[:orders].min() / np.linalg.norm(norms) > SHARE


def _flat(g, seed):
    return synth.geometric_spectrum(g.M, g.nrc, g.nz, g.nzc, seed=seed, a=1.0, b=1.0, c=0.8)


def _vector_reference(n, dealias):
    M = n // 2 + 1 - dealias
    g = Grid(M + 2, n, NZ, 0.8, lz=3.0, nphic=M)
    psi, chi, taps = _flat(g, 2), _flat(g, 3), {}
    rhs_tp(psi, chi, g, VecTables(g), U=(0.3, -0.2, 0.5), dealias=bool(dealias), taps=taps)
    return g, psi, chi, taps


def _orders(n, M, dealias):
    return min(M, (n + 1) // 2, (n - 1) // 3 + 1 if dealias else M)


@pytest.mark.parametrize("dealias", [0, 1])
@pytest.mark.parametrize("n", PAIRS)
def test_vector_stage(n, dealias):
    m = _gpu()
    print("orders, vector stage", n, dealias, flush=True)
    g, psi, chi, taps = _vector_reference(n, dealias)
    kept = _orders(n, g.M, dealias)
    for f in list(taps["u"]) + list(taps["w"]):
        assert _excited(np.moveaxis(np.fft.rfft(f, axis=-1), -1, 0), kept)
    plan = m.Plan(g.nr, n, NZ, 0.8, 3.0, nphic=g.M, dealias=dealias)
    tp, po, co = plan.taps_buffer(), plan.empty_spec(), plan.empty_spec()
    plan.rhs_tp(torch.from_numpy(to_lib(psi)).cuda(), torch.from_numpy(to_lib(chi)).cuda(), po, co, U=(0.3, -0.2, 0.5), taps=tp)
    got, pe = tp.cpu().numpy(), plan.layout.phys_elems
    nodal = got[:9 * pe].reshape(9, NZ, g.nr, n)
    for i, ref in enumerate(list(taps["u"]) + list(taps["w"]) + list(taps["N"])):
        assert rel(nodal[i], ref) < TOL, (i, rel(nodal[i], ref))
    src = got[9 * pe:].view(np.complex128).reshape(3, plan.tau, NZ)
    scale = max(np.linalg.norm(taps[k]) for k in "CKZ")
    for i, k in enumerate("CKZ"):
        assert np.linalg.norm(from_lib(src[i], g.M, g.nrc) - taps[k]) < TOL * scale, k
    # Zhat alone, order by order: the forward transform of N_z without cancellation
    mine = from_lib(src[2], g.M, g.nrc)
    assert _excited(taps["Z"], kept)
    assert rel(mine, taps["Z"]) < TOL


@pytest.mark.parametrize("n", PAIRS + WIDE)
def test_scalar_stages(n):
    m = _gpu()
    print("orders, scalar stages", n, flush=True)
    M = n // 2 + 1
    g = Grid(M + 1, n, 1, 0.9, nphic=M)
    t, S = Tables(g), _flat(g, 4)
    plan = m.Plan(g.nr, n, 1, 0.9, nphic=M, dealias=1)
    phys, spec = plan.empty_phys(), plan.empty_spec()
    plan.backward(torch.from_numpy(to_lib(S)).cuda(), phys)
    ref = backward(S, g, t)
    assert _excited(np.moveaxis(np.fft.rfft(ref, axis=-1), -1, 0), _orders(n, M, 0))
    assert rel(phys.cpu().numpy(), ref) < TOL
    plan.forward(phys, spec)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), forward(ref, g, t)) < TOL
    for kind, name in ((m.MLG_RHS_U2, "u2"), (m.MLG_RHS_KPP, "kpp")):
        plan.rhs_scalar(kind, 0.25, torch.from_numpy(to_lib(S)).cuda(), spec)
        ref = rhs_scalar(S, g, t, name, 0.25)
        assert _excited(ref, _orders(n, M, 1))
        assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < TOL


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_stages(prec):
    m = _gpu()
    print("orders, batch", prec, flush=True)
    sizes = [((n - 1) // 3 + 3, n) for n in SMOOTH]
    b = m.Batch([m.mlg_grid(nr, n, 1, 0, 0, 0, 1.0, 2 * np.pi, 1) for nr, n in sizes], prec=m.MLG_FP32 if prec else 0)
    sin, sout = b.empty_spec(), b.empty_spec()
    refs = []
    for k, (nr, n) in enumerate(sizes):
        g = Grid(nr, n, 1, 1.0)
        S = _flat(g, 90 + k)
        if prec:
            S = S.astype(np.complex64).astype(np.complex128)
        sin[int(b.offsets[k]):int(b.offsets[k + 1])] = torch.from_numpy(to_lib(S)[:, 0]).to(sin.dtype).cuda()
        refs.append((g, rhs_scalar(S, g, Tables(g), "kpp", 0.25)))
        assert _excited(refs[-1][1], _orders(n, g.M, 1)), n
    for cfg in ((1, 128, 8, 6), (0, 256, 8, 8)):
        b.set_config(*cfg)
        b.rhs_kpp(0.25, sin, sout)
        got = sout.cpu().numpy().astype(np.complex128)
        for k, (g, want) in enumerate(refs):
            mine = from_lib(got[int(b.offsets[k]):int(b.offsets[k + 1])][:, None], g.M, g.nrc)
            assert rel(mine, want) < (1e-5 if prec else TOL), (sizes[k], cfg, rel(mine, want))
    b.close()
