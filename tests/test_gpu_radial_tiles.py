"""Radial products of one field at the edges of their tiles (csrc/gemm_fold.hip, radial_gemm_f64) against the
oracle: odd N_r (a middle node, table rows of odd length), row tiles of 64 nodes or 128 pairs with remainders,
column tiles of 32 and 64, stages of 8 and 16 terms, launches below and above 512 blocks.

Tolerance: the parity bar of the FP64 paths (1e-12 normwise).
"""
import numpy as np
import pytest

from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.transform import Tables, backward, forward

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("case", [
    # nr, nphi, nz, nrc
    (2, 4, 2, 0), (3, 4, 3, 0), (33, 8, 16, 0), (64, 8, 18, 0), (65, 10, 15, 50), (127, 6, 36, 0), (129, 6, 8, 0),
    (130, 6, 9, 128), (257, 4, 20, 0), (260, 4, 20, 0), (63, 48, 180, 0), (64, 48, 180, 0),
])
def test_radial_tiles(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    nr, nphi, nz, nrc = case
    print("radial tiles", case, flush=True)
    g = Grid(nr, nphi, nz, 1.1, lz=2.5, nrc=nrc)
    t = Tables(g)
    plan = Plan(nr, nphi, nz, 1.1, 2.5, nrc=nrc)
    s = np.random.default_rng(nr).standard_normal((nz, nr, nphi))
    spec, back = plan.empty_spec(), plan.empty_phys()
    plan.forward(torch.from_numpy(s).cuda(), spec)
    ref = forward(s, g, t)
    assert rel(from_lib(spec.cpu().numpy(), g.M, g.nrc), ref) < 1e-12
    plan.backward(torch.from_numpy(to_lib(ref)).cuda(), back)
    assert rel(back.cpu().numpy(), backward(ref, g, t)) < 1e-12
