"""Columns of more than 1024 degrees (2D plans; the recurrence's coefficients as 32-bit whole numbers would overflow from
degree 1025), which take more than one chunk of the matrix-vector products (csrc/gemv.hip, the N_z = 1 step kernels) and five of the
pointwise evaluation.

* transforms against the oracle: 1e-12 normwise, the parity bar of the FP64 paths;
* steps against the same operators in tiles (the k = 0 slot of an N_z = 2 plan): both round the two products with V^-1 and V, whose
  condition is sqrt(n (n + 1) / 2) = 778 at 1100 degrees: 2 x 778 x sqrt(1100) x 1.1e-16 = 6e-12;
* pointwise values against the extended-precision recurrence: the chain of 1100 degrees, 1100 x 1.1e-16 x 2 of the largest sum.
"""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.basis import pbar
from oracle.grid import Grid
from oracle.transform import Tables, backward, forward

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    return Plan


@pytest.mark.parametrize("nr", [1025, 1026, 1100, 2100])
def test_products(nr):
    Plan = _gpu()
    print("long columns, products", nr, flush=True)
    g = Grid(nr, 4, 1, 1.2)
    t = Tables(g)
    plan = Plan(nr, 4, 1, 1.2)
    phys = np.random.default_rng(nr).standard_normal((1, nr, 4))
    spec, back = plan.empty_spec(), plan.empty_phys()
    plan.forward(torch.from_numpy(phys).cuda(), spec)
    ref = forward(phys, g, t)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < 1e-12
    plan.backward(torch.from_numpy(to_lib(ref)).cuda(), back)
    assert rel(back.cpu().numpy(), backward(ref, g, t)) < 1e-12


def test_steps():
    Plan = _gpu()
    print("long columns, steps", flush=True)
    nr = 1100
    flat, tiles = Plan(nr, 4, 1, 1.2), Plan(nr, 4, 2, 1.2)
    rng = np.random.default_rng(1)
    decay = np.concatenate([0.99 ** np.arange(nr - m) for m in range(flat.layout.M)])
    s, a1, a0 = ((rng.standard_normal(flat.tau) + 1j * rng.standard_normal(flat.tau)) * decay for _ in range(3))
    got = {}
    for nz, plan in ((1, flat), (2, tiles)):
        plan.step_setup(0.02, 1e-12, 4, 0.02)
        v = [torch.zeros((plan.tau, nz), dtype=torch.complex128, device="cuda") for _ in range(4)]
        for d, h in zip(v, (s, a1, a0)):
            d[:, 0] = torch.from_numpy(h).cuda()
        plan.step_abcn(v[0], v[1], v[2], v[3])
        got[nz, "abcn"] = v[3][:, 0].cpu().numpy()
        plan.step_febe(0, v[0], v[1], v[3])
        got[nz, "febe"] = v[3][:, 0].cpu().numpy()
    for k in ("abcn", "febe"):
        err = rel(got[1, k], got[2, k])
        print("  ", k, err, flush=True)
        assert err < 6e-12


@pytest.mark.parametrize("m", [0, 1])
def test_pointwise(m):
    Plan = _gpu()
    print("long columns, pointwise", m, flush=True)
    nr, ell = 1100, 1.2
    plan = Plan(nr, 4, 1, ell)
    rng = np.random.default_rng(2)
    spec = rng.standard_normal((plan.tau, 1)) + 1j * rng.standard_normal((plan.tau, 1))
    r = np.concatenate([[0.0], np.geomspace(1e-2, 1e2, 69)])
    out = plan.eval_harmonic(torch.from_numpy(spec).cuda(), m, 0, torch.from_numpy(r).cuda()).cpu().numpy().ravel()
    rl = r.astype(np.longdouble)
    x = (rl * rl - np.longdouble(ell) ** 2) / (rl * rl + np.longdouble(ell) ** 2)
    P = pbar(m, nr, x)[m:]
    col = spec[:nr, 0] if m == 0 else spec[nr:2 * nr - 1, 0]
    want = (P * col.real[:, None].astype(np.longdouble)).sum(0) + 1j * (P * col.imag[:, None].astype(np.longdouble)).sum(0)
    bound = nr * 1.1e-16 * 2 * np.abs(P * np.abs(col)[:, None]).sum(0).max()
    print("  error", np.abs(out - want).max(), "bound", bound, flush=True)
    assert np.abs(out - want).max() < bound
